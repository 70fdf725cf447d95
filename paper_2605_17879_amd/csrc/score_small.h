// Scoring of small columns (up to 4 096 ranks): one wave per column, one workgroup of M
// waves per step.  Included by score.hip, whose row functions it shares and whose launcher
// draws the line to the histogram route.
//
// A column of 1 024 values is sixteen registers of one wave.  The histogram route spends
// its time on fixed costs there (clearing, scanning and searching a thousand buckets, with
// 64 threads): 112 us for 1 024 ranks x 2 000 steps x 4 metrics, 25 us per step of which
// hardly anything is arithmetic.  Here the order statistics are found without LDS tables or
// barriers: the wave counts how many values lie under a pivot (a compare and a count of the
// lanes that answered, per register), two pivots at a time, first around the middle of a
// sorted sample of 64 values and then where the counts so far put the wanted rank; when at
// most 64 values are left between the pivots they are moved to one register and sorted by
// lane exchanges.  The scalar unit adds up the counts while the vector unit compares.
// Measured (launch): 1 024 x 2 000 x 4 112 -> 31 us, 1 000 x 1 x 4 (one step) 74 -> 9 us,
// 64 x 200 x 1 22 -> 4.4 us; 2 048 x 2 000 x 4 120 -> 49 us, 3 000 x 2 000 x 4 116 -> 66 us,
// 4 000 x 2 000 x 4 118 -> 88 us.  Bound by instruction issue in batches, by the length of the
// chain (load, median, MAD, scores) in one-step calls.
#ifndef GD_SCORE_SMALL_H_
#define GD_SCORE_SMALL_H_

// Rows: register rows of 64 x 4 ranks.  LDS of a workgroup, in this order, for M metrics.
template <int ROWS>
struct SmallLds {
    static constexpr int WORDS = ROWS * WAVE;        // exceed-mask words of a step
    uint64_t* node;        // [M][ROWS]   lane 2p: node p of the row exceeds
    uint32_t* exceed;      // [M][WORDS]  bit 0 of each byte: the rank exceeds
    uint32_t* slots;       // [M][64]     the wave's last candidates
    __device__ __forceinline__ SmallLds(unsigned char* raw, uint32_t M) {
        node = reinterpret_cast<uint64_t*>(raw);
        exceed = reinterpret_cast<uint32_t*>(raw + (size_t)M * ROWS * 8);
        slots = exceed + (size_t)M * WORDS;
    }
    static constexpr size_t bytes(uint32_t M) { return (size_t)M * (ROWS * 8 + WORDS * 4 + WAVE * 4); }
};

// Keys are worked out from the values whenever they are looked at: a second copy of the
// column would double its registers, and the optimiser is kept from making one by the
// token of each pass, a constant that it cannot see through.  Of a column without signs: its
// bits (missing samples, NaNs, lie above infinity, the largest key).
template <int ROWS>
struct PlainKeys {
    const float (&v)[ROWS][4];
    static constexpr uint32_t END = 0x7F800001u;
    __device__ __forceinline__ uint32_t token() const { return 0u; }
    __device__ __forceinline__ uint32_t at(int j, int i, uint32_t) const { return __float_as_uint(v[j][i]); }
    __device__ __forceinline__ float value(uint32_t k) const { return __uint_as_float(k); }
};
// Of any other: an order-preserving image, -0 reading as +0, NaNs above everything.
template <int ROWS>
struct MappedKeys {
    const float (&v)[ROWS][4];
    static constexpr uint32_t END = 0xFFFFFFFFu;
    __device__ __forceinline__ uint32_t token() const { return opaque_s(0u); }
    __device__ __forceinline__ uint32_t at(int j, int i, uint32_t zero) const {
        const float g = v[j][i] + __uint_as_float(zero);
        return g != g ? 0xFFFFFFFFu : key_of(g);
    }
    __device__ __forceinline__ float value(uint32_t k) const { return float_of_key(k); }
};
// Distances from the median.
template <int ROWS>
struct DistanceKeys {
    const float (&v)[ROWS][4];
    float med;
    static constexpr uint32_t END = 0x7F800001u;
    __device__ __forceinline__ uint32_t token() const { return opaque_s(__float_as_uint(med)); }
    __device__ __forceinline__ uint32_t at(int j, int i, uint32_t med_bits) const {
        return __float_as_uint(fabsf(v[j][i] - __uint_as_float(med_bits)));
    }
    __device__ __forceinline__ float value(uint32_t k) const { return __uint_as_float(k); }
};

// One key of every lane, from all rows.
template <int ROWS, typename Keys>
__device__ __forceinline__ uint32_t small_sample(const Keys& keys) {
    const uint32_t tok = keys.token();
    if constexpr (ROWS == 1) return keys.at(0, 0, tok);
    else if constexpr (ROWS == 2)
        return __builtin_amdgcn_inverse_ballot_w64(gd_lanes_with<32>()) ? keys.at(1, 0, tok) : keys.at(0, 0, tok);
    else {
        constexpr int STEP = ROWS / 4;
        const bool odd = __builtin_amdgcn_inverse_ballot_w64(gd_lanes_with<16>());
        const uint32_t lower = odd ? keys.at(STEP, 0, tok) : keys.at(0, 0, tok);
        const uint32_t upper = odd ? keys.at(3 * STEP, 0, tok) : keys.at(2 * STEP, 0, tok);
        return __builtin_amdgcn_inverse_ballot_w64(gd_lanes_with<32>()) ? upper : lower;
    }
}

// The order statistics k0 <= k1 <= k0 + 1 of the n keys below Keys::END among the wave's
// (the others, padding and missing samples, are END or above).  Throughout, clo keys lie
// under lo and chi under hi, with clo <= k0 and k1 < chi.  Ends for any contents: a round
// narrows [lo, hi) to a part of it, from the fourth on to a half.
// sort(sample): the sample's keys in ascending order (where n is more than a wave's).
template <int ROWS, typename Keys, typename Sort>
__device__ __forceinline__ void wave_select(const Keys& keys, uint32_t n, uint32_t k0, uint32_t k1, uint32_t lane,
                                            uint32_t* slots, uint32_t* s0, uint32_t* s1, Sort sort) {
    constexpr int V = ROWS * 4;
    uint32_t lo = 0, hi = Keys::END, clo = 0, chi = n;
    // two pivots, p <= q; true when one of them parts the two statistics (k0 < p <= k1)
    auto narrow = [&](uint32_t p, uint32_t q) -> bool {
        uint32_t cp = 0, cq = 0;
        const uint32_t tok = keys.token();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const uint32_t k = keys.at(i / 4, i % 4, tok);
            cp += (uint32_t)__popcll(gd_ballot(k < p));
            cq += (uint32_t)__popcll(gd_ballot(k < q));
        }
        uint32_t part = 0;
        bool parted = false;
        auto take = [&](uint32_t at, uint32_t c) {
            const bool up = c <= k0 && at > lo, down = c > k1 && at < hi, splits = c > k0 && c <= k1;
            lo = up ? at : lo; clo = up ? c : clo;
            hi = down ? at : hi; chi = down ? c : chi;
            part = splits ? at : part; parted = parted || splits;
        };
        take(p, cp);
        take(q, cq);
        if (parted) {
            uint32_t mx = 0, mn = 0xFFFFFFFFu;
            const uint32_t again = keys.token();
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const uint32_t k = keys.at(i / 4, i % 4, again);
                mx = max(mx, k < part ? k : 0u);
                mn = min(mn, k < part ? 0xFFFFFFFFu : k);
            }
            *s0 = (uint32_t)__builtin_amdgcn_readlane((int)wave_max_to_last(mx), WAVE - 1);
            *s1 = (uint32_t)__builtin_amdgcn_readlane((int)wave_min_to_last(mn), WAVE - 1);
        }
        return parted;
    };
    if (n > (uint32_t)WAVE) {
        // around the middle of the sample: two standard deviations of its median's rank
        // (and its middle value alone, where an eighth of the sample is that value: of few distinct
        // ones -- whole degrees -- it is mostly the one wanted)
        uint32_t mid = 0xFFFFFFFFu;
        const uint32_t sample = small_sample<ROWS>(keys);
        const uint32_t ns = (uint32_t)__popcll(gd_ballot(sample < Keys::END));
        if (ns >= 16) {
            const uint32_t sorted = sort(sample);
            const uint32_t reach = 4u + ns / 16u;
            const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(ns / 2 - reach));
            const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)min(ns / 2 + reach, ns - 1)) + 1u;
            const uint32_t m0 = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(ns / 2 - 4));
            const uint32_t m1 = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(ns / 2 + 3));
            mid = m0 == m1 ? m0 : mid;
            if (narrow(p, q)) return;
        }
        for (int round = 0; chi - clo > (uint32_t)WAVE; ++round) {
            const uint32_t span = hi - lo;
            if (span <= 1) { *s0 = lo; *s1 = lo; return; }             // ties
            uint32_t p = span / 2, q = p;
            if (mid != 0xFFFFFFFFu) {
                p = mid > lo ? mid - lo : 0u;
                q = p + 1u;
                mid = 0xFFFFFFFFu;
            } else if (round < 3) {
                // the values between the pivots taken as evenly spread: the wanted rank's
                // place, and 2.5 standard deviations of it to either side
                const float c = (float)(chi - clo), at = (float)(k1 - clo) + 0.5f;
                const float side = 4.0f + 1.25f * __builtin_sqrtf(c), scale = (float)span / c;
                p = (uint32_t)fminf(fmaxf((at - side) * scale, 0.0f), 4294967040.0f);
                q = (uint32_t)fminf(fmaxf((at + side) * scale, 0.0f), 4294967040.0f);
            }
            p = rfl(min(max(p, 1u), span - 1u));
            q = rfl(min(max(q, 1u), span - 1u));
            if (narrow(lo + p, lo + q)) return;
        }
    }
    // at most 64 keys in [lo, hi)
    const uint32_t width = hi - lo;
    const uint32_t tok = keys.token();
    uint32_t pos = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t k = keys.at(i / 4, i % 4, tok);
        const bool hit = k - lo < width;
        const uint64_t mask = gd_ballot(hit);
        if (mask != 0ull) {
            // (chi - clo of them by the counts, so that every place is one of the wave's 64)
            const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, pos));
            if (hit) slots[to] = k;
            pos += (uint32_t)__popcll(mask);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // (an infinite median leaves fewer distances than n: slots that no lane wrote are not read)
    const uint32_t c = gd_sort64(lane < pos ? slots[lane] : 0xFFFFFFFFu);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    *s0 = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)((k0 - clo) & (WAVE - 1)));
    *s1 = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)((k1 - clo) & (WAVE - 1)));
}

// multi-signal rule on four mask bytes at once: primary bit set and at least min_signals
// bits in the byte; the answer is bit 0 of each byte
__device__ __forceinline__ uint32_t small_rule4(uint32_t E, uint32_t primary, uint32_t min_signals) {
    uint32_t pc = E - ((E >> 1) & 0x55555555u);
    pc = (pc & 0x33333333u) + ((pc >> 2) & 0x33333333u);
    pc = (pc + (pc >> 4)) & 0x0F0F0F0Fu;
    return ((E >> primary) & 0x01010101u) & ((pc + (0x80u - min_signals) * 0x01010101u) >> 7);
}

// FULL: R == ROWS * 256.  A workgroup for every step (no loop over steps: the compiler
// would keep the sorts' lane masks in scalar registers across it, and spill them).
template <int ROWS, bool FULL, bool WANT_Z>
__device__ __forceinline__ void score_small(const gd_score_args& a) {
    constexpr int V = ROWS * 4;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const uint32_t R = a.R, N = a.N, M = a.M, RW = (R + 63) / 64, NWD = (N + 63) / 64;
    const SmallLds<ROWS> lds(lds_raw, M);
    const uint32_t lane = threadIdx.x & (WAVE - 1), m = rfl(threadIdx.x / WAVE);
    const float thr = a.thr;
    uint32_t dir_codes = 0;          // direction + 1 of metric i in bits 2i, 2i + 1
#pragma unroll
    for (int i = 0; i < 8; ++i) dir_codes |= (uint32_t)(a.dir[i] + 1) << (2 * i);
    const int dir = (int)(rfl(dir_codes) >> (2u * m) & 3u) - 1;
    const size_t t = blockIdx.x;
    const size_t column = t * M + m;
    const float* col = a.x + column * R;
    auto holds = [&](int j) { return FULL || j * 256 + lane * 4 < R; };
    float v[ROWS][4];
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        float4 q = make_float4(__uint_as_float(0x7FFFFFFFu), __uint_as_float(0x7FFFFFFFu),
                               __uint_as_float(0x7FFFFFFFu), __uint_as_float(0x7FFFFFFFu));     // padding
        if (holds(j)) q = *reinterpret_cast<const float4*>(col + j * 256 + lane * 4);
        v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    }
    // the lane's largest bit pattern: signs, missing samples (NaN) and magnitudes
    uint32_t um = 0;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const uint32_t rm = max(max(__float_as_uint(v[j][0]), __float_as_uint(v[j][1])),
                                max(__float_as_uint(v[j][2]), __float_as_uint(v[j][3])));
        um = max(um, holds(j) ? rm : 0u);
    }
    const bool special = gd_ballot(um > 0x7F800000u) != 0ull, signs = gd_ballot(um >= 0x80000000u) != 0ull;
    uint32_t present = R;
    if (special) {
        present = 0;
#pragma unroll
        for (int i = 0; i < V; ++i) present += (uint32_t)__popcll(gd_ballot(v[i / 4][i % 4] == v[i / 4][i % 4]));
    }
    float med = __uint_as_float(0x7FC00000u), mad = med;             // nothing to take a median of
    if (present) {
        const uint32_t k0 = (present - 1) / 2, k1 = present / 2;
        uint32_t* const slots = lds.slots + m * WAVE;
        uint32_t s0, s1;
        float rising = 0.0f;                    // the median's sample in ascending order
        // (an odd count has one middle value: no sum that could overflow)
        if (!signs) {
            const PlainKeys<ROWS> keys{v};
            wave_select<ROWS>(keys, present, k0, k1, lane, slots, &s0, &s1, [&](uint32_t sample) {
                const uint32_t sorted = gd_sort64(sample);
                rising = keys.value(sorted);
                return sorted;
            });
            med = k0 == k1 ? keys.value(s0) : 0.5f * (keys.value(s0) + keys.value(s1));
        } else {
            const MappedKeys<ROWS> keys{v};
            wave_select<ROWS>(keys, present, k0, k1, lane, slots, &s0, &s1, [&](uint32_t sample) {
                const uint32_t sorted = gd_sort64(sample);
                rising = keys.value(sorted);
                return sorted;
            });
            med = k0 == k1 ? keys.value(s0) : 0.5f * (keys.value(s0) + keys.value(s1));
        }
        // The MAD's sample holds the same values: in their order their distances fall and then rise (missing
        // ones at the end, made alike), and the last six of a sort's 21 stages are what remains of it
        // (with that, and three instructions less for each candidate's place, 1 024 ranks x 2 000 x 4
        // 30.0 -> 29.0 us, one step of 1 000 x 4 10.35 -> 9.93).
        const DistanceKeys<ROWS> keys{v, med};
        wave_select<ROWS>(keys, present, k0, k1, lane, slots, &s0, &s1, [&](uint32_t) {
            const float d = fabsf(rising - med);
            return gd_merge<64, false>(d == d ? __float_as_uint(d) : 0xFFFFFFFFu);
        });
        mad = k0 == k1 ? keys.value(s0) : 0.5f * (keys.value(s0) + keys.value(s1));
    }
    if (lane == 0) { a.med[column] = med; a.mad[column] = mad; }
    float s = 1.4826f * mad;
    s = fmaxf(s, a.rel_floor * fabsf(med));
    s = fmaxf(s, a.abs_floor);
    // (as in score_columns: the quotient by the reciprocal is exact in this range)
    const bool exact_recip = !special && gd_ballot(um > 0x5D000000u) == 0ull && med >= 0x1p-34f &&
                             s >= 0x1p-60f && s <= 0x1p60f;
    const float r1 = 1.0f / s;
    if (WANT_Z) {
        float* zcol = a.z + column * R;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            float q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = v[j][i];
                if (exact_recip) {
                    const float d = x - med;
                    const float q0 = d * r1;
                    const float e0 = __builtin_fmaf(-q0, s, d);
                    const float q1 = __builtin_fmaf(e0, r1, q0);
                    const float e1 = __builtin_fmaf(-q1, s, d);
                    q[i] = __builtin_fmaf(e1, r1, q1);
                } else {
                    q[i] = x == x ? ((x + 0.0f) - med) / s : 0.0f;       // a missing sample scores 0
                }
            }
            if (holds(j)) *reinterpret_cast<float4*>(zcol + j * 256 + lane * 4) = make_float4(q[0], q[1], q[2], q[3]);
        }
    }
    const float ss = dir < 0 ? -s : s, rs = dir < 0 ? -r1 : r1;
    const uint32_t absmask = dir == 0 ? 0x7FFFFFFFu : 0xFFFFFFFFu, sgnmask = dir < 0 ? 0x80000000u : 0u;
    const bool fast = exact_recip && a.node_agg == 0;
    float* nzrow = a.node_z + t * N;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        uint32_t e;
        float nz;
        if (fast && dir != 0) score_row_fast<false>(v[j], med, ss, rs, thr, a.node_scale, 0x01010101u, &e, &nz);
        else if (fast) score_row_fast<true>(v[j], med, ss, rs, thr, a.node_scale, 0x01010101u, &e, &nz);
        else score_row(a.node_agg, v[j], med, s, absmask, sgnmask, thr, a.node_scale, &e, &nz);
        lds.exceed[m * SmallLds<ROWS>::WORDS + j * WAVE + lane] = e;
        const uint64_t nb = gd_ballot(nz > thr);
        if (lane == 0) lds.node[m * ROWS + j] = nb;
        if (m == a.primary && holds(j) && !(lane & 1)) nzrow[(j * 256 + lane * 4) / 8] = nz;
    }
    __syncthreads();
    // The step's mask bytes and anomaly words: row c of 64 mask words per wave.
    for (uint32_t c = m; c < (uint32_t)ROWS; c += M) {
        const uint32_t q = c * WAVE + lane;
        const bool valid = q * 4 < R;
        uint32_t E = 0;
        for (uint32_t i = 0; i < M; ++i) E |= lds.exceed[i * SmallLds<ROWS>::WORDS + q] << i;
        if (valid) reinterpret_cast<uint32_t*>(a.exceed_mask + t * R)[q] = E;
        const uint32_t an = valid ? small_rule4(E, a.primary, a.min_signals) : 0u;
        const uint32_t nib = (an | (an >> 7) | (an >> 14) | (an >> 21)) & 0xFu;
        const uint32_t sub = lane & 15;
        uint32_t wlo = sub < 8 ? nib << (4 * sub) : 0u, whi = sub >= 8 ? nib << (4 * (sub - 8)) : 0u;
        wlo |= gd_lane_xor<1>(wlo, lane); whi |= gd_lane_xor<1>(whi, lane);
        wlo |= gd_lane_xor<2>(wlo, lane); whi |= gd_lane_xor<2>(whi, lane);
        wlo |= gd_lane_xor<4>(wlo, lane); whi |= gd_lane_xor<4>(whi, lane);
        wlo |= gd_lane_xor<8>(wlo, lane); whi |= gd_lane_xor<8>(whi, lane);
        if (sub == 0 && valid) a.rank_anom[t * RW + q / 16] = ((uint64_t)whi << 32) | wlo;
    }
    for (uint32_t c = M - 1 - m; c < NWD; c += M) {              // (the waves with no row above first)
        const uint32_t n = c * WAVE + lane;
        uint32_t b = 0;
        if (n < N)
            for (uint32_t i = 0; i < M; ++i)
                b |= (uint32_t)(lds.node[i * ROWS + n / 32] >> (2 * (n % 32)) & 1ull) << i;
        if (n < N) a.node_mask[t * N + n] = (uint8_t)b;
        const uint64_t word = gd_ballot(((b >> a.primary) & 1u) && (uint32_t)__popc(b) >= a.min_signals);
        if (lane == 0) a.node_anom[t * NWD + c] = word;
    }
}

#endif  // GD_SCORE_SMALL_H_
