// Scoring kernel: per (step, metric) cross-rank median and MAD by selection,
// robust z, exceedance, multi-signal combine and 8-GPU node scores
// (Section 4.2 peer-relative evaluation and multi-signal rule; Section 7.1
// 8-GPU nodes).
//
// Persistent workgroups: each takes a contiguous run of steps and scores them
// column after column.  For each of a step's M columns it
//   1. holds the column in registers (float4 per lane per row, loaded once from
//      HBM, coalesced, rank-contiguous; the next column is loaded row by row
//      while the current one is scored) -- a column is never read again, but for the
//      rows asked for ahead (five or six in two tilings) where the column before
//      them leaves the hinted route and they are not kept;
//   2. finds the two middle order statistics by counting: a bracket (taken from
//      the previous step of the same metric, else from a sample of the column)
//      is counted into an LDS histogram of order-preserving integer keys, a
//      scan locates the bucket(s) holding the wanted ranks, a second pass
//      gathers that bucket's few values into LDS where they are ranked exactly;
//      a bracket that misses, or a bucket that is too full (ties), falls back
//      to wider or narrower ranges until the answer is exact;
//   3. gets the MAD from the same histogram (bucket edges on either side of the median bound the
//      wanted distances, and the values there are gathered in the same pass or in one of their
//      own), or by a second selection on |x - med| when that does not apply;
//   4. computes z, the exceedance bits and the node scores from the registers.
// After the M columns the per-rank mask bytes, anomaly bits and node outputs
// are written.  HBM traffic is the 4 bytes per sample read plus ~1.8 bytes per
// rank and step of outputs.
#include <type_traits>

#include "gd_bracket.h"
#include "gd_grant.h"
#include "gd_internal.h"
#include "gd_lanes.h"
#include "gd_sample.h"

// This file is compiled several times, side by side: as it is (every launch without the
// optional z output, and the entry points), through score_z.hip with GD_SCORE_WANT_Z = 1
// (the launches that write z as well), and through the score_ragged files with
// GD_SCORE_RAGGED = 1, 2 or 3 (the rank counts that fill no tiling exactly).
#ifndef GD_SCORE_WANT_Z
#define GD_SCORE_WANT_Z 0
#endif
#ifndef GD_SCORE_RAGGED
#define GD_SCORE_RAGGED 0
#endif

namespace {

constexpr bool WANT_Z_HERE = GD_SCORE_WANT_Z != 0;

constexpr int WAVE = 64;
constexpr int CAND_CAP = 512;  // values ranked exactly in LDS per selection

// (of a condition as it is: __ballot takes an integer, and makes one first)
__device__ __forceinline__ uint64_t gd_ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ uint32_t rfl(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return __uint_as_float(rfl(__float_as_uint(v))); }

// Order-preserving map fp32 -> u32 and back.
__device__ __forceinline__ uint32_t key_of(float f) {
    uint32_t b = __float_as_uint(f);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float float_of_key(uint32_t k) {
    uint32_t b = (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
    return __uint_as_float(b);
}

// Ranks whose exceed bits one workgroup of combine_kernel puts together.
constexpr uint32_t PLANE_RANKS = 2048;

// What the score loop needs to know of a column (worked out by one wave).
struct alignas(16) ScoreParams {
    float s, ss, rs;           // scale, its signed form and the reciprocal of that
    float cc, kk, margin;          // node estimate of the decision-only route
    uint32_t scut, xcut;           // and its bounds, for `decided`
    uint32_t route, exact_recip;
    float med, mad;
    uint32_t settled;              // the gathered candidates gave median and MAD
};
// What the first wave works these out from: the same for all columns.
struct alignas(16) ScoreRules {
    float thr, node_scale, rel_floor, abs_floor;
    float inv_node_scale;
    uint32_t agg;
};

// What the hinted selection gathers (worked out by one wave).  Buckets are of its counting pass.
struct alignas(16) GatherPlan {
    // the MAD's buckets, lb0 .. li - 1 left of the median and rb0 .. rx - 1 right of it: what lies
    // between them is nearer to `center` than `inner`, or in them; n_in values there, n_out with theirs
    float inner;
    uint32_t li, rb0, n_in;
    float outer;                   // what lies beyond them is farther from `center`
    uint32_t lb0, rx, n_out;
    float center, reach;           // |x - center| <= reach: in one of the median's buckets,
    uint32_t mid, status;          // the first in the low half, further ones in the high half; PLAN_*
    uint32_t lo, shift;            // bucket b starts at the key lo + (b << shift)
    uint32_t skip, n_mid;          // values before the median's buckets and in them
};
constexpr uint32_t PLAN_NONE = 0, PLAN_LOCATED = 1, PLAN_GATHER = 2;
// Gathered at the most.  sh.cand holds the ones, the others and a wave's worth of room for the last
// of them; these words are CAND_NONE (above every key, and a NaN) between columns.
constexpr uint32_t MOST_MID = 64, MOST_DIST = 256, CAND_REST = MOST_MID + MOST_DIST + WAVE, CAND_NONE = 0x7FFFFFFFu;
static_assert(CAND_REST <= (uint32_t)CAND_CAP, "the gathered candidates fit their list");
// Buckets from the one that holds the lower middle rank to the upper one's: the two are neighbours, so
// that nothing lies in those between.  (One in twenty columns of 5 000 ranks, where a bucket holds
// a value or two, has them further apart than one, and a batch is done when its slowest column
// is: 5 000 x 1 000 x 2 41 us a launch where these went the general way, 29.5 so, 8 000 x 1 000 x 4
// 81 and 52.  A launch of 16 384 x 10 000 x 4 differs by less than with the place of its buffers: 515 to 605.)
constexpr uint32_t MOST_APART = 63;

template <int NT, int LOG_NB, int MAX_NODES>
struct Shared {
    static constexpr int NB = 1 << LOG_NB, WAVES = NT / WAVE;
    // dlo, hist, dhi are one array of 64 + NB + 64 counters for the hinted counting pass
    // (keys under / inside / over the bracket); the other passes use hist alone.
    uint32_t dlo[64];
    uint32_t hist[NB];
    uint32_t dhi[64];
    uint32_t pref[NB + 4];     // exclusive prefix sums of hist (pref[NB] = total), for the MAD shortcut
    alignas(16) uint32_t cand[CAND_CAP + 4];   // read four at a time when ranking
    uint32_t wpart[16];
    uint32_t below, ncand;
    uint32_t nkept, nnear;     // hinted MAD: candidates kept after the exact test, and those found nearer
    uint32_t smin, smax;       // extremes of the sample keys
    uint32_t d1, d2;           // MAD shortcut: distance interval holding the wanted ranks
    uint32_t umax[2];          // largest raw bit pattern of the column (double-buffered)
    uint32_t res[6];           // ba, prefix before ba, bb, prefix through bb, va, vb
    // Per metric, from the previous step scored by this workgroup: the median and how
    // far below / above it the counting histogram reached (hok = the hint is usable).
    float hmed[8], hwl[8], hwh[8], hmad[8];
    uint32_t hok[8];
    uint32_t hfast[8];         // the hinted selection below has not failed for this metric yet
    ScoreParams par;
    ScoreRules rules;
    GatherPlan plan;
    alignas(8) uint8_t nodeb[MAX_NODES];        // the step's node mask bytes, read eight at a time
    uint64_t ranka[MAX_NODES / 8 > 0 ? MAX_NODES / 8 : 1];     // the step's rank anomaly words (zero between steps)
};

// Cross-lane moves with immediate patterns (DPP): no address registers, nothing
// for the optimiser to hoist out of the column loop.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {   // lanes without a source read 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
}
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp1(uint32_t v) {   // lanes without a source read all ones
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, ROW_MASK, 0xF, false);
}
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
    else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
    else if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);
    else {
        static_assert(J == 4, "lane_xor");
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (J << 10));
    }
}
__device__ __forceinline__ float lane_xor1(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0xB1, 0xF, 0xF, true));
}

// Inclusive prefix sum across the wave (lane 63 ends with the total).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += dpp0<0x111>(v);          // row_shr:1
    v += dpp0<0x112>(v);          // row_shr:2
    v += dpp0<0x114>(v);          // row_shr:4
    v += dpp0<0x118>(v);          // row_shr:8
    v += dpp0<0x142, 0xA>(v);     // row_bcast:15 into rows 1 and 3
    v += dpp0<0x143, 0xC>(v);     // row_bcast:31 into rows 2 and 3
    return v;
}
// Minimum / maximum over the wave, valid in lane 63 (lanes without a source read what changes
// nothing, so that a step is one instruction).
__device__ __forceinline__ uint32_t wave_min_to_last(uint32_t v) {
    v = min(v, dpp1<0x111>(v)); v = min(v, dpp1<0x112>(v));
    v = min(v, dpp1<0x114>(v)); v = min(v, dpp1<0x118>(v));
    v = min(v, dpp1<0x142, 0xA>(v)); v = min(v, dpp1<0x143, 0xC>(v));
    return v;
}
__device__ __forceinline__ uint32_t wave_max_to_last(uint32_t v) {
    v = max(v, dpp0<0x111>(v)); v = max(v, dpp0<0x112>(v));
    v = max(v, dpp0<0x114>(v)); v = max(v, dpp0<0x118>(v));
    v = max(v, dpp0<0x142, 0xA>(v)); v = max(v, dpp0<0x143, 0xC>(v));
    return v;
}

// Exclusive prefix sum of one value per thread over the workgroup; total in *tot.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t tid, uint32_t* wpart,
                                                    uint32_t* tot) {
    const uint32_t lane = tid & (WAVE - 1), w = tid >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == WAVE - 1) wpart[w] = inc;
    __syncthreads();
    // every wave scans the (at most 16) wave totals itself: one LDS read, a row scan
    uint32_t p = lane < (uint32_t)(NT / WAVE) ? wpart[lane] : 0u;
    p += dpp0<0x111>(p); p += dpp0<0x112>(p); p += dpp0<0x114>(p); p += dpp0<0x118>(p);
    const uint32_t total = __builtin_amdgcn_readlane((int)p, NT / WAVE - 1);
    const uint32_t wu = rfl(w);
    const uint32_t off = wu ? (uint32_t)__builtin_amdgcn_readlane((int)p, (int)(wu - 1)) : 0u;
    *tot = total;
    return off + inc - v;
}

// Loads and stores of what passes through once (the telemetry; mask bytes and z, written in whole
// lines), marked as such: memory takes them sooner.  A pass of 16 384 ranks x 10 000 x 4 693 us
// without the marks, 654 with those of the loads, 646 with the masks' too; 65 536 x 4 096 x 8 2 054,
// 2 001, 1 990; 40 000 x 1 024 x 8 416, 410, 408; 32 768 x 512 x 8 with z 266 and 255.  (The node
// bytes, and the columns of one wave, are no faster with them; the ledger's reads are slower, 118 and
// 122 us: it finds part of the masks in the last cache.)
typedef float gd_f4 __attribute__((ext_vector_type(4)));
typedef uint32_t gd_u4 __attribute__((ext_vector_type(4)));
constexpr int NONTEMPORAL = 2;            // (of a buffer load's cache policy)
__device__ __forceinline__ void store_once(float* p, float x, float y, float z, float w) {
    const gd_f4 q = {x, y, z, w};
    __builtin_nontemporal_store(q, reinterpret_cast<gd_f4*>(p));
}
__device__ __forceinline__ void store_once(uint32_t* p, uint32_t v) { __builtin_nontemporal_store(v, p); }

// Values the optimiser cannot see through.  They stop it from keeping one
// pass's per-element temporaries, or values derived from the thread index,
// alive in registers across the whole column loop.
__device__ __forceinline__ uint32_t opaque_s(uint32_t v) {   // wave-uniform
    v = rfl(v);
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ uint32_t opaque_v(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Keys of the median selection.  PLAIN: the column has no sign bit set, so the
// raw bits order like the values; otherwise the order-preserving image is used.
template <int ROWS, bool PLAIN>
struct XKeys {
    const float (&v)[ROWS][4];
    __device__ __forceinline__ uint32_t token() const { return opaque_s(31u); }
    __device__ __forceinline__ uint32_t key(float f, uint32_t tok) const {
        if (PLAIN) return __float_as_uint(f);
        // -0 reads as +0; the zero is derived from the opaque token so that the
        // sum is recomputed per pass instead of being kept for all 64 values
        const float g = f + __uint_as_float(tok - 31u);
        const uint32_t b = __float_as_uint(g);
        const uint32_t k = b ^ ((uint32_t)((int32_t)b >> tok) | 0x80000000u);   // tok is an opaque 31
        return g != g ? 0xFFFFFFFFu : k;     // a missing sample (NaN) lies above every value
    }
    __device__ __forceinline__ uint32_t at(int j, int i, uint32_t tok) const { return key(v[j][i], tok); }
    __device__ __forceinline__ float value(uint32_t k) const {
        return PLAIN ? __uint_as_float(k) : float_of_key(k);
    }
};

// Keys of the MAD selection: the bits of |x - med| (non-negative floats order as integers).
template <int ROWS>
struct DKeys {
    const float (&v)[ROWS][4];
    float med;
    __device__ __forceinline__ uint32_t token() const { return opaque_s(__float_as_uint(med)); }
    __device__ __forceinline__ uint32_t key(float f, uint32_t tok) const {
        return __float_as_uint(fabsf(f - __uint_as_float(tok)));     // tok is an opaque med
    }
    __device__ __forceinline__ uint32_t at(int j, int i, uint32_t tok) const { return key(v[j][i], tok); }
    __device__ __forceinline__ float value(uint32_t k) const { return __uint_as_float(k); }
};

// LDS protocol of the selection code.  Between uses the work area is kept in a
// known state, so that no phase has to clear it behind two barriers of its own:
// sh.hist all zero (locate() clears what it reads), sh.below = sh.ncand = 0,
// sh.smin = ~0, sh.smax = 0, sh.d1 = 0, sh.d2 = ~0.  Thread 0 restores a scalar
// after the barrier that follows its last read, and at least one more barrier
// precedes the next atomic update of it.

// After a counting pass: find the buckets holding ranks ka and kb (relative to
// everything; `sh.below` keys lie under the histogram's range, or none if
// !USE_BELOW).  Clears the histogram, leaves the results in sh.res, returns the
// below count and whether both ranks fall inside the histogram.  Ends with a barrier.
template <int NT, int LOG_NB, bool WRITE_PREF, bool USE_BELOW, typename SH>
__device__ __forceinline__ bool locate(SH& sh, uint32_t tid, uint32_t ka, uint32_t kb,
                                       uint32_t* below_out) {
    constexpr int BPT = (1 << LOG_NB) / NT;
    uint32_t loc[BPT], s = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) { loc[q] = sh.hist[tid * BPT + q]; s += loc[q]; }
#pragma unroll
    for (int q = 0; q < BPT; ++q) sh.hist[tid * BPT + q] = 0;
    uint32_t total;
    const uint32_t excl = block_excl_scan<NT>(s, tid, sh.wpart, &total);
    const uint32_t below = USE_BELOW ? sh.below : 0u;
    const uint32_t ra = ka - below, rb = kb - below;   // wrap when not bracketed
    if (WRITE_PREF) {
        uint32_t p = excl;
#pragma unroll
        for (int q = 0; q < BPT; ++q) { sh.pref[tid * BPT + q] = p; p += loc[q]; }
        if (tid == NT - 1) sh.pref[1 << LOG_NB] = p;
    }
    if (ra - excl < s) {
        uint32_t p = excl;
        bool done = false;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (!done && ra - p < loc[q]) { sh.res[0] = tid * BPT + q; sh.res[1] = p; done = true; }
            p += loc[q];
        }
    }
    if (rb - excl < s) {
        uint32_t p = excl;
        bool done = false;
#pragma unroll
        for (int q = 0; q < BPT; ++q) {
            if (!done && rb - p < loc[q]) { sh.res[2] = tid * BPT + q; sh.res[3] = p + loc[q]; done = true; }
            p += loc[q];
        }
    }
    __syncthreads();
    if (USE_BELOW && tid == 0) sh.below = 0;
    *below_out = rfl(below);
    return rfl(ka >= below && rb < total) != 0;
}

// A wave's own list of register rows (four values of a lane) that hold a value somebody looks
// for.  Rows instead of values, at a position made of a count in a scalar register and the
// lanes' ballot: six instructions for the rows with a hit, and no round trip to LDS; which of
// the four values it was is found out afterwards, by drain(), a value per lane.  The list lies in
// the counters, which are at rest between two counting passes, and leaves them at rest.  Room for
// more rows, or a second walk for those that did not fit, is no gain: crowded buckets are ranked
// then instead of narrowed, and to rank a few hundred candidates takes longer (16 384 ranks x 2 048 x
// 2, 400 equal values about the median: 189 us; 866 with a second walk, which costs plain columns
// 1 to 2 % too).
template <typename SH, uint32_t MOST_ROWS = 64>
struct RowList {
    static constexpr uint32_t MOST = MOST_ROWS;    // rows of a wave
    static_assert(MOST * 4 * SH::WAVES <= SH::NB, "the waves' lists lie in the counters");
    uint32_t* const words;
    uint32_t n = 0;                                // (wave-uniform)
    __device__ __forceinline__ RowList(SH& sh, uint32_t w) : words(sh.hist + w * (MOST * 4u)) {}
    __device__ __forceinline__ bool overflow() const { return n > MOST; }
    __device__ __forceinline__ void add(bool hit, const float (&row)[4]) {
        const uint64_t hm = gd_ballot(hit);
        if (__builtin_expect(hm != 0ull, 0)) {
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, n));
            if (hit) {
                // (two words at a time: a store of all four ties the row's registers together, and the
                // column is then copied between passes; a list that is full overwrites itself)
                uint32_t* const to = words + 4 * (pos & (MOST - 1));
#pragma unroll
                for (int i = 0; i < 4; i += 2)
                    __hip_atomic_store(reinterpret_cast<uint64_t*>(to + i), (uint64_t)__float_as_uint(row[i + 1]) << 32 | __float_as_uint(row[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
            n += (uint32_t)__popcll(hm);
        }
    }
    // use(value, valid) for every value listed, by whole waves
    template <typename Use>
    __device__ __forceinline__ void drain(uint32_t lane, Use use) {
        const uint32_t end = 4u * min(n, MOST);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t at = 0; at < end; at += WAVE) {
            const bool valid = at + lane < end;
            uint32_t x = 0;
            if (valid) { x = words[at + lane]; words[at + lane] = 0; }
            use(x, valid);
        }
        n = 0;
    }
};

// The lanes with a hit append their value to a list shared by the workgroup (whole waves call).
__device__ __forceinline__ void append(uint32_t lane, uint32_t* list, uint32_t* count, bool hit, uint32_t value) {
    const uint64_t hm = gd_ballot(hit);
    if (hm == 0ull) return;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(count, (uint32_t)__popcll(hm));
    base = rfl(base);
    const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, base));
    if (hit && to < (uint32_t)CAND_CAP) list[to] = value;
}

// The keys in [clo, clo + cspan], no more than CAND_CAP, one by one into sh.cand: where a wave's list
// of rows was too short for them (buckets of few candidates, most of them one wave's: 200 of 48 000
// ranks x 1 024 steps 155 us where the whole column was selected anew, 104 so).  Begins and ends
// with a barrier.
template <int ROWS, typename SH, typename Keys>
__device__ __forceinline__ void gather_singly(SH& sh, const Keys& keys, uint32_t clo, uint32_t cspan) {
    __syncthreads();                        // everyone has read the lists' count
    if (threadIdx.x == 0) sh.ncand = 0;
    __syncthreads();
    const uint32_t tok = keys.token(), from = opaque_s(clo);
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        uint32_t off[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) off[i] = keys.at(j, i, tok) - from;
        if (min(min(off[0], off[1]), min(off[2], off[3])) <= cspan) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (off[i] <= cspan) {
                    const uint32_t pos = atomicAdd(&sh.ncand, 1u);
                    if (pos < (uint32_t)CAND_CAP) sh.cand[pos] = off[i] + from;
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
}

// Exact ranking of the cnt gathered candidates in sh.cand: those of rank wa and wb go to
// sh.res[4] and sh.res[5].  Up to a wave's worth each wave takes every (NT/64)-th candidate; its lanes
// split the comparisons and the wave counts the lanes that answered yes (ties broken by position).
// More of them: a lane takes a candidate and goes through the others, which the waves of the
// same 64 candidates share; the counts (fewer, and not more) meet in the histogram, which is
// at rest and left so.  (With a wave to a candidate there too, a read from LDS to wait for in
// every 64 comparisons: 200 alike values about the median in one wave's ranks, 20 000 ranks x 1 000
// 58.8 us, so 46.9.)  Ends with a barrier.
template <int NT, typename SH>
__device__ __forceinline__ void rank_candidates(SH& sh, uint32_t tid, uint32_t cnt, uint32_t wa, uint32_t wb) {
    const uint32_t* const list = sh.cand;
    const uint32_t lane = tid & (WAVE - 1), w = rfl(tid >> 6);
    if (cnt <= (uint32_t)WAVE) {
        // one LDS read per wave: lane j holds candidate j, candidate i is read from lane i
        // (read whatever the slot holds: the load then does not wait for cnt)
        const uint32_t cj = list[lane];
        for (uint32_t i = w; i < cnt; i += NT / WAVE) {
            const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)cj, (int)i);
            const uint32_t r = (uint32_t)__popcll(gd_ballot(lane < cnt && (cj < c || (cj == c && lane < i))));
            if (lane == 0) {
                if (r == wa) sh.res[4] = c;
                if (r == wb) sh.res[5] = c;
            }
        }
    } else {
        constexpr uint32_t WAVES = NT / WAVE;
        const uint32_t groups = (cnt + WAVE - 1) / WAVE, parts = groups < WAVES ? WAVES / groups : 1u, fours = cnt / 4;
        for (uint32_t u = w; u < groups * parts; u += WAVES) {
            const uint32_t g = u % groups, part = u / groups, i = g * WAVE + lane;
            const uint32_t mine = list[i];               // (below CAND_CAP, whatever it holds beyond the last)
            uint32_t fewer = 0, upto = 0;                // candidates below this one, and not above it
            auto compare = [&](uint32_t other) {
                fewer += other < mine ? 1u : 0u;
                upto += other <= mine ? 1u : 0u;
            };
            const uint32_t end = fours * (part + 1) / parts;
            for (uint32_t at = fours * part / parts; at < end; ++at) {
                const uint4 q = reinterpret_cast<const uint4*>(list)[at];
                compare(q.x); compare(q.y); compare(q.z); compare(q.w);
            }
            if (part == 0)
                for (uint32_t j = 4 * fours; j < cnt; ++j) compare(list[j]);
            if (i < cnt) atomicAdd(&sh.hist[i], upto << 16 | fewer);
        }
        __syncthreads();
        for (uint32_t i = tid; i < cnt; i += NT) {
            const uint32_t r = sh.hist[i], c = list[i];
            sh.hist[i] = 0;
            if ((r & 0xFFFFu) <= wa && wa < r >> 16) sh.res[4] = c;      // (alike ones write the same)
            if ((r & 0xFFFFu) <= wb && wb < r >> 16) sh.res[5] = c;
        }
    }
    __syncthreads();
}

// Exact selection of the order statistics k0 <= k1 (0-based, k1 - k0 <= 1) of
// the ROWS*4 keys per thread held in registers (padding keys compare above all
// real ones).
//   1. One sampled key per thread (skey, svalid; n of them valid) goes into a histogram over the
//      sample's own range; the sample ranks n/2 -+ 2*sqrt(n) give a bracket
//      [lo, hi] that holds the wanted ranks with high probability and only a
//      small share of the column.
//   2. Counting pass: keys inside the bracket go into the LDS histogram, keys
//      below it are counted.  If the wanted ranks are not inside, count again
//      over the full range.
//   3. The buckets holding the ranks are gathered into LDS and ranked exactly,
//      or, when they are crowded (ties), the range is narrowed to the bucket.
//
// WIDE: bracket the sample ranks n/2 -+ 0.34*n instead, so that the histogram also
// covers the values around median -+ MAD, and keep its prefix sums in sh.pref.  If
// the first counting pass settles the selection, *hist_lo / *hist_shift describe
// that histogram (bucket b holds keys hist_lo + b*2^shift ...) and the function
// returns true; the MAD shortcut then reads the prefix sums.
//
// umax_slot (with a handed-in bracket only): the first counting pass also finds the
// largest raw bit pattern of the column and leaves it in *umax_out.  Should it carry
// a sign bit or be a NaN's, the raw bits were no valid keys or the ranks asked for
// not the right ones: the selection stops after clearing its work area and the
// caller starts over.
template <int NT, int ROWS, int LOG_NB, bool WIDE, typename SH, typename Keys>
__device__ __forceinline__ bool block_select(SH& sh, const Keys& keys, uint32_t skey, bool svalid,
                                             uint32_t n, uint32_t k0, uint32_t k1, uint32_t* out0,
                                             uint32_t* out1, uint32_t* hist_lo = nullptr,
                                             uint32_t* hist_hi = nullptr, int* hist_shift = nullptr,
                                             bool hinted = false, uint32_t hint_lo = 0,
                                             uint32_t hint_hi = 0, uint32_t* umax_slot = nullptr,
                                             uint32_t* umax_out = nullptr) {
    constexpr int NB = 1 << LOG_NB;
    constexpr int BPT = NB / NT;
    static_assert(BPT >= 1 && (BPT % 4 == 0 || BPT < 4), "bucket split");
    // What is gathered singly where the lists are too short: as much as sixteen waves rank sooner than
    // the next round of counting would narrow; four or eight waves rank little (12 000 ranks x 1 000
    // x 2, 150 equal values about the median: 162 us narrowed, 201 ranked).
    constexpr uint32_t MOST_SINGLY = NT >= 1024 ? CAND_CAP : 2 * RowList<SH>::MOST;
    uint32_t lo = hint_lo, hi = hint_hi;
    // Bracket from the sample (skipped while a bracket handed in by the caller holds).
    auto sample_bracket = [&]() {
        const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1);
        const uint32_t mn = wave_min_to_last(svalid ? skey : 0xFFFFFFFFu);
        const uint32_t mx = wave_max_to_last(svalid ? skey : 0u);
        if (lane == WAVE - 1) { atomicMin(&sh.smin, mn); atomicMax(&sh.smax, mx); }
        __syncthreads();
        const uint32_t smin = rfl(sh.smin), smax = rfl(sh.smax);
        const uint32_t sspan = smax - smin;                 // smin <= smax: some sample is valid
        const int sshift = shift_for<LOG_NB>(sspan);
        if (svalid) atomicAdd(&sh.hist[(skey - smin) >> sshift], 1u);
        __syncthreads();
        if (tid == 0) { sh.smin = 0xFFFFFFFFu; sh.smax = 0; }
        // n valid samples: the ranks n/2 -+ (2*sqrt(n) + 1) bracket the column's median
        const uint32_t delta = WIDE ? (n * 87u) >> 8 : (uint32_t)(2.0f * __builtin_sqrtf((float)n)) + 1u;
        const uint32_t half = n / 2;
        const uint32_t ra = half > delta ? half - 1 - delta : 0u;
        const uint32_t rb = min(n - 1, half + delta);
        uint32_t unused;
        const bool both = locate<NT, LOG_NB, false, false>(sh, tid, ra, rb, &unused);
        const uint32_t ba = rfl(sh.res[0]), bb = rfl(sh.res[2]);
        lo = ra == 0 ? 0u : smin + (ba << sshift);
        const uint64_t hend = (uint64_t)smin + ((uint64_t)(bb + 1) << sshift) - 1;
        hi = rb == n - 1 ? 0xFFFFFFFFu : (hend > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)hend);
        // Fewer samples than n went in when some were missing values: a sample rank
        // beyond them was not located, and the bracket is then left open.
        if (!both) { lo = 0; hi = 0xFFFFFFFFu; }
    };
    if (!hinted) sample_bracket();
    // mode 0: both statistics together; 1: k0 alone; 2: k1 alone (after a split)
    int mode = 0, rounds = 0;
    uint32_t ka = k0, kb = k1, v0 = 0, v1 = 0;
    for (;;) {
        ++rounds;
        const uint32_t span = hi - lo;
        const int shift = shift_for<LOG_NB>(span);
        // a fresh copy of the thread index per round: values derived from it (bucket
        // slots, LDS addresses) are then recomputed instead of living in registers
        const uint32_t tid = opaque_v(threadIdx.x);
        const uint32_t lane = tid & (WAVE - 1);
        // counting pass
        uint32_t nbelow = 0;   // per lane; summed over the wave after the pass
        const bool with_umax = umax_slot != nullptr && rounds == 1;
        uint32_t um = 0;
        {
            const uint32_t tok = keys.token();
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t kk = keys.at(j, i, tok);
                    nbelow += kk < lo ? 1u : 0u;
                    const uint32_t t = kk - lo;
                    if (t <= span) atomicAdd(&sh.hist[t >> shift], 1u);
                }
                if (umax_slot != nullptr) {     // (padding lanes never take this route: FULL tilings only)
                    // the row's registers are made opaque here, or the maxima, which do not
                    // depend on the round, are all computed ahead of the loop -- after
                    // waiting for the whole column instead of row by row
                    float(&row)[4] = const_cast<float(&)[4]>(keys.v[j]);
                    asm volatile("" : "+v"(row[0]), "+v"(row[1]), "+v"(row[2]), "+v"(row[3]));
                    um = max(um, max(keys.at(j, 0, tok), keys.at(j, 1, tok)));
                    um = max(um, max(keys.at(j, 2, tok), keys.at(j, 3, tok)));
                    asm volatile("" : "+v"(um));
                }
                asm volatile("" : "+v"(nbelow));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        nbelow = wave_incl_scan(nbelow);
        if (with_umax) um = wave_max_to_last(um);
        if (lane == WAVE - 1) {
            if (nbelow) atomicAdd(&sh.below, nbelow);
            if (with_umax) atomicMax(umax_slot, um);
        }
        __syncthreads();
        if (with_umax) {
            const uint32_t umax = rfl(*umax_slot);
            *umax_out = umax;
            if (umax > 0x7F800000u) {
                uint32_t unused;
                (void)locate<NT, LOG_NB, false, true>(sh, tid, ka, kb, &unused);   // clears the work area
                *out0 = 0; *out1 = 0;
                return false;
            }
        }
        uint32_t below;
        const bool bracketed = locate<NT, LOG_NB, WIDE, true>(sh, tid, ka, kb, &below);
        if (!bracketed) {
            // the bracket missed: a handed-in one is replaced by the sample's, the
            // sample's by the full key range
            if (hinted) { hinted = false; sample_bracket(); }
            else { lo = 0; hi = 0xFFFFFFFFu; __syncthreads(); }
            continue;
        }
        const uint32_t ba = rfl(sh.res[0]), pa = rfl(sh.res[1]);
        const uint32_t bb = rfl(sh.res[2]), pb = rfl(sh.res[3]);
        uint32_t va = lo + ba, vb = lo + bb;            // shift == 0: one key per bucket, the answer
        bool settled = shift == 0;
        if (!settled && pb - pa <= (uint32_t)CAND_CAP) {
            // gather the values of buckets ba..bb and rank them exactly
            const uint32_t clo = lo + (ba << shift);
            const uint64_t cend = (uint64_t)lo + ((uint64_t)(bb + 1) << shift) - 1;
            const uint32_t chi = cend > hi ? hi : (uint32_t)cend;
            const uint32_t cspan = chi - clo;
            const uint32_t tok = keys.token();
            RowList<SH> rows(sh, rfl(tid >> 6));
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
                // one test per register row (hits are rare): the smallest offset decides
                uint32_t off[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) off[i] = keys.at(j, i, tok) - clo;
                rows.add(min(min(off[0], off[1]), min(off[2], off[3])) <= cspan, keys.v[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
            rows.drain(lane, [&](uint32_t x, bool valid) {
                const uint32_t kk = keys.key(__uint_as_float(x), tok);
                append(lane, sh.cand, &sh.ncand, valid && kk - clo <= cspan, kk);
            });
            __syncthreads();
            const uint32_t cnt = pb - pa;
            settled = rfl(sh.ncand) == cnt;             // (else a wave's list was too short)
            if (!settled && cnt <= MOST_SINGLY) {
                gather_singly<ROWS>(sh, keys, clo, cspan);
                settled = true;
            }
            if (settled) {
                rank_candidates<NT>(sh, tid, cnt, ka - below - pa, kb - below - pa);
                va = rfl(sh.res[4]); vb = rfl(sh.res[5]);
            } else {
                __syncthreads();
            }
            if (tid == 0) sh.ncand = 0;
        }
        if (!settled) {
            // crowded (ties): look inside bucket ba; if the two statistics sit in
            // different crowded buckets, finish k0 first, then k1 on its own
            if (ba != bb) { mode = 1; kb = ka; }
            const uint32_t nlo = lo + (ba << shift);
            const uint64_t nend = (uint64_t)nlo + ((uint64_t)1 << shift) - 1;
            hi = nend > hi ? hi : (uint32_t)nend;
            lo = nlo;
            __syncthreads();
            continue;
        }
        if (mode == 0) {
            v0 = va; v1 = vb;
            if (WIDE && hist_lo) { *hist_lo = lo; *hist_hi = hi; *hist_shift = shift; }
            break;
        }
        if (mode == 1) {
            v0 = va; mode = 2; ka = kb = k1; lo = 0; hi = 0xFFFFFFFFu;
            __syncthreads();
            continue;
        }
        v1 = va;
        break;
    }
    *out0 = v0;
    *out1 = v1;
    return rounds == 1 && mode == 0;
}

// MAD shortcut for a sign-free column whose median selection left a histogram of
// the raw bits over [lo, hi] (2^shift keys per bucket, prefix sums in sh.pref)
// that reaches well beyond median -+ MAD.  From the prefix sums alone the threads
// find a distance interval [d1, d2] that must hold the wanted order statistics of
// |x - med| (see below); one pass then counts the distances below d1 exactly and
// gathers those inside the interval (a few dozen) for exact ranking.  The pass
// also verifies the interval; false is returned, and the caller selects in the
// ordinary way, if the histogram did not reach far enough or the check fails.
template <int NT, int ROWS, int LOG_NB, typename SH>
__device__ __forceinline__ bool mad_from_histogram(SH& sh, const float (&v)[ROWS][4], float med,
                                                   uint32_t lo, uint32_t hi, int shift, uint32_t k0,
                                                   uint32_t k1, float mad_hint, uint32_t* out0,
                                                   uint32_t* out1) {
    constexpr int NB = 1 << LOG_NB;
    const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1);
    const float xlo = __uint_as_float(lo), xhi = __uint_as_float(hi);
    const float dmax = fminf(med - xlo, xhi - med);
    if (!(dmax > 0.0f) || shift < 2) return false;
    // With the previous step's MAD of this metric as a hint only the edges whose
    // distance from the median is within an eighth of it are paired (a couple of
    // hundred, one per thread); if they do not enclose the ranks, all edges are.
    uint32_t d1 = 0, d2 = 0;
    auto grid = [&](bool near_hint_only) -> bool {
        // Pairs of bucket edges (eL, eR) with value(eL) <= med < value(eR): the set
        // S = {eL <= key < eR} is counted exactly by the prefix sums, every value
        // outside S is at least min(dL, dR) away from med and every value inside at
        // most max(dL, dR) (subtraction is monotone), where dL = med - value(eL) and
        // dR = value(eR) - med.  So |S| <= k0 makes min(dL, dR) a valid d1 and
        // |S| >= k1 + 1 makes max(dL, dR) a valid d2.  Each thread pairs its own
        // buckets' edges with the two edges that nearly mirror them.
        constexpr int BPT = NB / NT;
        uint32_t c1 = 0, c2 = 0xFFFFFFFFu;
        auto edge = [&](uint32_t b) { return __uint_as_float(lo + (b << shift)); };
        const uint32_t bmax = (hi - lo) >> shift;     // last bucket whose lower edge is <= hi
        auto eval = [&](uint32_t bL, uint32_t bR) {
            if (bL < bR && bR <= bmax) {
                const float xl = edge(bL), xr = edge(bR);
                if (xl <= med && xr > med) {
                    const float dl = med - xl, dr = xr - med;
                    const uint32_t cntS = sh.pref[bR] - sh.pref[bL];
                    if (cntS <= k0) c1 = max(c1, __float_as_uint(fminf(dl, dr)));
                    if (cntS >= k1 + 1) c2 = min(c2, __float_as_uint(fmaxf(dl, dr)));
                }
            }
        };
        auto pair_edge = [&](uint32_t b) {
            const float xe = edge(b);
            if (xe > med) {            // a right edge: mirror it to the left
                const uint32_t km = __float_as_uint(med - (xe - med));
                if (km >= lo && km <= hi) {
                    const uint32_t bl = (km - lo) >> shift;
                    eval(bl, b);
                    eval(bl + 1, b);
                }
            } else {                   // a left edge: mirror it to the right
                const uint32_t km = __float_as_uint(med + (med - xe));
                if (km >= lo && km <= hi) {
                    const uint32_t br = (km - lo) >> shift;
                    eval(b, br);
                    eval(b, br + 1);
                }
            }
        };
        if (near_hint_only) {
            // the edges within an eighth of the hint around med - hint and med + hint,
            // dealt out one per thread
            const float wl0 = med - 1.125f * mad_hint, wl1 = med - 0.875f * mad_hint;
            const float wr0 = med + 0.875f * mad_hint, wr1 = med + 1.125f * mad_hint;
            const uint32_t klo = __float_as_uint(fmaxf(wl0, xlo)), khi = __float_as_uint(fminf(wr1, xhi));
            const uint32_t bl0 = (klo - lo) >> shift, bl1 = (__float_as_uint(fmaxf(wl1, xlo)) - lo) >> shift;
            const uint32_t br0 = (__float_as_uint(fminf(wr0, xhi)) - lo) >> shift, br1 = (khi - lo) >> shift;
            // (at most NB edges a side whatever the hint and the bounds hold -- infinities, NaN
            // patterns, a window turned inside out: the loop below stays short, and eval()
            // checks every bucket index against bmax before it reads a prefix sum)
            const uint32_t nl = min(bl1 - bl0 + 1, (uint32_t)NB), nr = min(br1 - br0 + 1, (uint32_t)NB);
            for (uint32_t e = tid; e < nl + nr; e += NT) pair_edge(e < nl ? bl0 + e : br0 + (e - nl));
        } else {
#pragma unroll
            for (int q = 0; q < BPT; ++q) pair_edge(tid * BPT + q);
        }
        c1 = wave_max_to_last(c1);
        c2 = wave_min_to_last(c2);
        if (lane == WAVE - 1) { atomicMax(&sh.d1, c1); atomicMin(&sh.d2, c2); }
        __syncthreads();
        d1 = rfl(sh.d1); d2 = rfl(sh.d2);
        if (d2 != 0xFFFFFFFFu && d2 >= d1) return true;
        __syncthreads();                     // everyone has read d1, d2
        if (tid == 0) { sh.d1 = 0; sh.d2 = 0xFFFFFFFFu; }
        return false;
    };
    bool found = mad_hint > 0.0f && grid(true);
    if (!found) {
        if (mad_hint > 0.0f) __syncthreads();    // the reset above precedes the next proposals
        found = grid(false);
    }
    if (!found) return false;
    // exact pass: count |x - med| below d1, gather those in [d1, d2]
    const uint32_t span = d2 - d1;
    uint32_t nbelow = 0;
    {
        const uint32_t tok = opaque_s(__float_as_uint(med));
        RowList<SH> rows(sh, rfl(tid >> 6));
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            uint32_t off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t kk = __float_as_uint(fabsf(v[j][i] - __uint_as_float(tok)));
                nbelow += kk < d1 ? 1u : 0u;
                off[i] = kk - d1;
            }
            // one test per register row (hits are rare): the smallest offset decides
            rows.add(min(min(off[0], off[1]), min(off[2], off[3])) <= span, v[j]);
            asm volatile("" : "+v"(nbelow));
            __builtin_amdgcn_sched_barrier(0);
        }
        if (rows.overflow() && lane == 0) atomicAdd(&sh.ncand, (uint32_t)CAND_CAP + 1u);
        rows.drain(lane, [&](uint32_t x, bool valid) {
            const uint32_t kk = __float_as_uint(fabsf(__uint_as_float(x) - __uint_as_float(tok)));
            append(lane, sh.cand, &sh.ncand, valid && kk - d1 <= span, kk);
        });
    }
    nbelow = wave_incl_scan(nbelow);
    if (lane == WAVE - 1 && nbelow) atomicAdd(&sh.below, nbelow);
    __syncthreads();
    if (tid == 0) { sh.d1 = 0; sh.d2 = 0xFFFFFFFFu; }
    const uint32_t below = rfl(sh.below), cnt = rfl(sh.ncand);
    if (cnt > (uint32_t)CAND_CAP || below > k0 || k1 >= below + cnt) {
        __syncthreads();                     // everyone has read the counters
        if (tid == 0) { sh.below = 0; sh.ncand = 0; }
        return false;
    }
    const uint32_t wa = k0 - below, wb = k1 - below;
    rank_candidates<NT>(sh, tid, cnt, wa, wb);
    if (tid == 0) { sh.below = 0; sh.ncand = 0; }
    *out0 = rfl(sh.res[4]);
    *out1 = rfl(sh.res[5]);
    return true;
}

// Hinted selection: median and MAD of a sign-free column whose predecessor (the same
// metric one step earlier) left a bracket around its median that reaches past median -+ MAD,
// and its MAD.  Two passes over the registers instead of the four of the general route:
//   1. counting: every key adds one to a counter -- its bucket inside the bracket, or a
//      lane-private word under / over it (no test, no branch: the bucket index is clamped);
//      the pass also finds the largest bit pattern of the column.
//   2. gathering.  The prefix sums give the median to a bucket or two, and with them the buckets
//      on either side that the middle distances may end in (plan_gather); one pass lists the
//      register rows that hold a value of any of these, and the waves sort out which.
// Then one wave takes the median from its bucket's values, classifies the others by their exact
// distances and takes the MAD (finish_gather); the values between the two ranges of the MAD's buckets
// are known from the prefix sums, so nothing is counted per value.  Where that fails -- crowded
// buckets, a list that is too short, a hint of the MAD that is far off -- the median's bucket is
// gathered and ranked by itself, the edges are searched for with the exact median and a third
// pass gathers what lies about them (hinted_rest).
// What bounds it: 16 waves of one workgroup a CU wait for the chain between the passes, in which a
// lone wave starts an instruction every eight cycles; so as few steps, and instructions, as can be.
// One gathering pass instead of two, and one wave instead of all for what comes after: 65 536 ranks x
// 4 096 x 8 a pass 1 974 -> 1 919 us (19.7 -> 17.9 vector and 8.8 -> 6.7 scalar instructions a
// sample), 40 000 x 1 024 x 8 381 -> 371, 32 768 x 512 x 8 with z 249 -> 245, one step of 32 768 x 8
// 27.8 -> 27.4; 16 384 x 10 000 x 4, four workgroups a CU, the same.  (With the candidates sorted by
// lane exchanges and kept unnarrowed that wave took 4 900 cycles a column instead of 3 800, and the
// gain was 0.2 %.)
// The result of either is exact: what lies between the buckets is nearer than DI, what lies beyond
// them farther than DO, and what is ranked in [DI, DO] must hold the ranks asked for.  The work
// area is at rest in every case, the column is never modified.
struct HintedResult {
    int found;                  // 2: median and MAD, 1: median alone
    uint32_t m0, m1;            // the two middle keys
    uint32_t q0, q1;            // the two middle distances (bit patterns), or, of `listed` ones in
    uint32_t listed;            // sh.cand (at most 64), their ranks: for the first wave to sort
};
struct GatherResult {
    uint32_t status;            // PLAN_*
    uint32_t umax;              // largest raw bit pattern of the column, of the samples that arrived
                                // where the median's buckets were found
    uint32_t present;           // samples that arrived, where some did not (0: all did)
};

// How many of the column's values are no NaNs, and their largest bit pattern (of a column
// without sign bits).  The work area is at rest before and after; two barriers.
template <int ROWS, typename SH>
__device__ __forceinline__ void count_present(SH& sh, const float (&v)[ROWS][4], uint32_t* present, uint32_t* top) {
    const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1);
    // (tested on the bit patterns, against an opaque constant: other tests of the same
    // registers must not be merged with these and kept for later)
    const uint32_t absm = opaque_s(0x7FFFFFFFu);
    uint32_t np = 0, um = 0;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t b = __float_as_uint(v[j][i]);
            const bool here = (b & absm) <= 0x7F800000u;
            np += here ? 1u : 0u;
            um = max(um, here ? b : 0u);
        }
        asm volatile("" : "+v"(np), "+v"(um));
        __builtin_amdgcn_sched_barrier(0);
    }
    np = wave_incl_scan(np);
    um = wave_max_to_last(um);
    if (lane == WAVE - 1) { atomicAdd(&sh.ncand, np); atomicMax(&sh.smax, um); }
    __syncthreads();
    *present = rfl(sh.ncand);
    *top = rfl(sh.smax);
    __syncthreads();                    // everyone has read them
    if (tid == 0) { sh.ncand = 0; sh.smax = 0; }
}

// What the hinted selection gathers, worked out by one wave from the prefix sums of the counting
// pass.  The median is known to its buckets ba..bb alone, ml <= median < mh, and so are the MAD's.
// Candidate e is a right edge (a bucket's lower edge, e > bb + 1); its distance from the median
// mirrored to the left gives an edge f, the first one above the mirror point, and F = #[f, e) never
// decreases with e.  It is taken for both ends of the median's range: Fl >= F >= Fh.  With the
// last e of Fl <= k0 at most k0 values are nearer than any value from f on outwards, with the first
// of Fh > k1 more than k1 are no farther; the wanted distances end in between.  The candidates looked
// at are the 64 edges around the one that the hint points at, one a lane; should they not hold the
// answer, every sixteenth of the 1 024 about them and then the 64 where those point (a hint that
// is 17 % off).  A wave that runs alone starts an instruction every eight cycles, of whatever kind
// (measured), so that the number of instructions counts here: what is not the lanes' is left to
// those who read the plan.
template <int LOG_NB, typename SH>
__device__ __forceinline__ void plan_gather(SH& sh, uint32_t lane, uint32_t lo, int shift, float mad_hint,
                                            uint32_t below, uint32_t k0, uint32_t k1) {
    constexpr uint32_t bmax = (1u << LOG_NB) - 1u;
    const uint32_t ba = rfl(sh.res[0]), pa = rfl(sh.res[1]);
    const uint32_t bb = rfl(sh.res[2]), pb = rfl(sh.res[3]);
    auto edge = [&](uint32_t e) { return __uint_as_float(lo + (e << shift)); };
    const float ml = edge(ba), mh = edge(bb + 1u), center = 0.5f * (ml + mh);
    GatherPlan& plan = sh.plan;
    if (lane == 0) {
        plan.center = center;
        plan.reach = fmaxf(center - ml, mh - center);
        plan.mid = ba | (bb - ba) << 16;
        // crowded (ties): the general route narrows
        plan.status = pb - pa > (uint32_t)CAND_CAP / 2 || bb - ba > MOST_APART ? PLAN_NONE : PLAN_LOCATED;
        plan.lo = lo; plan.shift = (uint32_t)shift; plan.skip = below + pa; plan.n_mid = pb - pa;
    }
    if (pb - pa > MOST_MID || bb - ba > MOST_APART || !(mad_hint > 0.0f)) return;
    // the first lane's edge (mod 2^32; a hint beyond the bracket points at its end)
    uint32_t e0 = rfl(min((__float_as_uint(center + mad_hint) - lo) >> shift, bmax)) - 32u;
    uint32_t step = 1;
    for (int round = 0; round < 3; ++round) {
        const uint32_t e = e0 + lane * step;
        const float x = edge(e);
        const uint32_t ql = (__float_as_uint(ml - (x - ml)) - lo) >> shift;      // (under the bracket: beyond bmax)
        const uint32_t qh = (__float_as_uint(mh - (x - mh)) - lo) >> shift;
        const float inner = fminf(center - edge(qh + 1u), edge(e - 1u) - center), outer = fmaxf(center - edge(ql), x - center);
        uint32_t pe = 0, pl1 = 0, ph = 0, pb1 = 0, cl = 0xFFFFFFFFu, ch = 0;
        if (e - (bb + 2u) < bmax - bb && ql <= bmax && qh < ba) {          // (e in bb + 2 .. bmax + 1)
            pe = sh.pref[e]; ph = sh.pref[qh + 1u]; pl1 = sh.pref[ql]; pb1 = sh.pref[e - 1u];
            cl = pe - sh.pref[ql + 1u];
            ch = pe - ph;
        }
        const uint64_t under = gd_ballot(cl <= k0), over = gd_ballot(ch > k1);
        if (round == 1) {                                          // the fine look, about where the coarse one points
            if (over == 0ull || under == 0ull) break;
            e0 += 16u * (63u - (uint32_t)__builtin_clzll(under)) - 24u;
            step = 1;
            continue;
        }
        if (over == 0ull || under == 0ull) {                       // not here: every sixteenth edge, 512 to either side
            e0 -= 32u * 15u;
            step = 16;
            continue;
        }
        // At most as many values as are asked for are closer than f, the edge that the last `under` gives
        // on the left.  Buckets grow wider with their values, so that f's own mirror image lies in the
        // bucket before the right edge.  (A bucket further in on both sides has twice as many distances
        // to rank where the left ones are narrow: exponential values, 56 000 ranks x 1 024 143 us, so 112.)
        if (lane == 63u - (uint32_t)__builtin_clzll(under)) {
            plan.inner = inner; plan.li = qh + 1u; plan.rb0 = e - 1u; plan.n_in = pb1 - ph;
            plan.status = inner > 0.0f ? PLAN_GATHER : PLAN_LOCATED;
        }
        if (lane == (uint32_t)__builtin_ctzll(over)) {
            plan.outer = outer; plan.lb0 = ql; plan.rx = e; plan.n_out = pe - pl1;
        }
        break;
    }
}

// The rank of one of N keys (N = 16, 32 or 64; no two of them alike but for the CAND_NONE that
// follow the last), by one wave: lane l ranks key l mod N, the lanes that rank the same one compare
// it with their share of the others each.  Two instructions a comparison, 28 in all for sixteen
// keys, 48 for thirty-two (a sort by lane exchanges takes seven for each of its ten to
// twenty-one steps).
template <int N>
__device__ __forceinline__ uint32_t rank_key(const uint32_t* list, uint32_t mine, uint32_t lane) {
    constexpr int SHARE = N * N / WAVE;
    const uint4* others = reinterpret_cast<const uint4*>(list + lane / N * SHARE);
    uint32_t r = 0;
#pragma unroll 1
    for (int at = 0; at < SHARE / 4; at += 2) {                  // (eight at a time: registers)
        uint32_t bits = 0;
#pragma unroll
        for (int i = 0; i < (SHARE < 8 ? SHARE / 4 : 2); ++i) {
            const uint4 q = others[at + i];
            auto smaller = [&](uint32_t other) { bits = __builtin_amdgcn_alignbit(bits, other - mine, 31); };      // (the difference's sign follows)
            smaller(q.x); smaller(q.y); smaller(q.z); smaller(q.w);
        }
        r += (uint32_t)__popc(bits);
    }
    if constexpr (N <= 32) {
        const auto h = __builtin_amdgcn_permlane32_swap(r, r, false, false);
        r = h[0] + h[1];
    }
    if constexpr (N <= 16) {
        const auto h = __builtin_amdgcn_permlane16_swap(r, r, false, false);
        r = h[0] + h[1];
    }
    return r;
}
// The keys of rank ka and kb among a list's first n, by one wave.
__device__ __forceinline__ void pick_ranks(const uint32_t* list, uint32_t n, uint32_t lane, uint32_t ka, uint32_t kb, uint32_t* a, uint32_t* b) {
    uint32_t mine, r;
    if (n <= 16) { mine = list[lane & 15]; r = rank_key<16>(list, mine, lane); }
    else if (n <= 32) { mine = list[lane & 31]; r = rank_key<32>(list, mine, lane); }
    else { mine = list[lane]; r = rank_key<64>(list, mine, lane); }
    *a = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(__builtin_ctzll(gd_ballot(r == ka)) & (WAVE - 1)));
    *b = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)(__builtin_ctzll(gd_ballot(r == kb)) & (WAVE - 1)));
}

// Median and MAD from what was gathered, by one wave: false where a wave's list was too short, or the
// ranks asked for are not among the candidates.  A candidate's distance is compared with the bounds
// inside which every value between the MAD's buckets lies and beyond which every value further out
// does, so that what is ranked is exact whatever the plan was.
template <typename SH>
__device__ __forceinline__ bool finish_gather(SH& sh, uint32_t lane, uint32_t k0, uint32_t k1, float* med_out, float* mad_out) {
    constexpr uint32_t CHUNKS = MOST_DIST / WAVE;
    static_assert(CHUNKS == 4, "two chunks, and two more");
    const GatherPlan plan = sh.plan;
    const uint32_t got = sh.ncand;
    uint32_t* const dist = sh.cand + MOST_MID;
    float d[CHUNKS];
#pragma unroll
    for (uint32_t c = 0; c < CHUNKS; ++c) d[c] = __uint_as_float(dist[c * WAVE + lane]);      // (none: a NaN)
    const uint32_t n_mid = rfl(plan.n_mid), n_in = rfl(plan.n_in), n_dist = rfl(plan.n_out) - n_in, skip = rfl(plan.skip);
    const uint32_t lo = rfl(plan.lo), shift = rfl(plan.shift);
    const bool whole = rfl(got) == (n_mid << 16 | n_dist), many = n_dist > 2 * WAVE;
    auto edge = [&](uint32_t e) { return __uint_as_float(lo + (e << shift)); };
    uint32_t s0, s1;
    pick_ranks(sh.cand, n_mid, lane, k0 - skip, k1 - skip, &s0, &s1);
    const uint32_t none = opaque_v(CAND_NONE), first = lo + ((rfl(plan.mid) & 0xFFFFu) << shift);
    sh.cand[lane] = none; dist[lane] = none; dist[WAVE + lane] = none;
    if (many) { dist[2 * WAVE + lane] = none; dist[3 * WAVE + lane] = none; }
    if (lane == 0) sh.ncand = opaque_v(0u);
    if (!whole) return false;
    const float med = 0.5f * (__uint_as_float(first + (s0 >> 6)) + __uint_as_float(first + (s1 >> 6)));
    float from = uniform(fmaxf(med - edge(plan.li), edge(plan.rb0) - med)), to = uniform(fminf(med - edge(plan.lb0), edge(plan.rx) - med));
#pragma unroll
    for (uint32_t c = 0; c < CHUNKS; ++c) d[c] = fabsf(d[c] - med);
    uint32_t nearer = 0, upto = 0;              // candidates nearer than `from`, and not beyond `to`
    auto count = [&](float x) {
        nearer += (uint32_t)__popcll(gd_ballot(x < from));
        upto += (uint32_t)__popcll(gd_ballot(x <= to));
    };
    auto classify = [&]() {
        nearer = 0; upto = 0;
        count(d[0]); count(d[1]);
        if (many) { count(d[2]); count(d[3]); }
    };
    classify();
    for (int round = 0; upto - nearer > 32u && round < 4; ++round) {
        // the candidates taken as evenly spread: the wanted rank's place, and 13 ranks to either side (the
        // one wanted among 64 is off by four, one standard deviation, at the most).  Beside that, the
        // search goes on with what lies on the rank's side.
        const float per = (to - from) * __builtin_amdgcn_rcpf((float)(upto - nearer)), at = from + (float)(int)(k0 - n_in - nearer) * per;
        const float first_from = from, first_to = to;
        const uint32_t first_nearer = nearer, first_upto = upto;
        from = uniform(fmaxf(from, at - 13.0f * per)); to = uniform(fminf(to, at + 13.0f * per));
        classify();
        if (__builtin_expect(n_in + nearer > k0, 0)) {
            to = __uint_as_float(__float_as_uint(from) - 1u); upto = nearer;
            from = first_from; nearer = first_nearer;
        } else if (__builtin_expect(k1 >= n_in + upto, 0)) {
            from = __uint_as_float(__float_as_uint(to) + 1u); nearer = upto;
            to = first_to; upto = first_upto;
        }
    }
    const uint32_t c_in = n_in + nearer, kept = upto - nearer, base = __float_as_uint(from);
    // (also where `from` is beyond `to`; keys of 25 bits and the place)
    if (c_in > k0 || k1 >= c_in + kept || kept > (uint32_t)WAVE || __float_as_uint(to) - base >= 1u << 25) return false;
    uint32_t* const slots = dist + MOST_DIST;
    uint32_t pos = 0;
    auto keep = [&](float x) {
        const uint32_t off = __float_as_uint(x) - base;
        const bool hit = off <= __float_as_uint(to) - base;
        const uint64_t mask = gd_ballot(hit);
        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, pos));
        if (hit) slots[at] = off << 6 | at;
        pos += (uint32_t)__popcll(mask);
    };
    keep(d[0]); keep(d[1]);
    if (many) { keep(d[2]); keep(d[3]); }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint32_t d0, d1;
    pick_ranks(slots, kept, lane, k0 - c_in, k1 - c_in, &d0, &d1);
    slots[lane] = none;
    *med_out = med;
    const float m0 = __uint_as_float(base + (d0 >> 6)), m1 = __uint_as_float(base + (d1 >> 6));
    *mad_out = k0 == k1 ? m0 : 0.5f * (m0 + m1);
    return true;
}

// Padding lanes (of the last rows of a ragged rank count) hold another lane's value until
// `set_padding(j)` makes them NaN patterns: over the bracket in the count, never within a
// distance in the gather.
// `counted` is called by every wave as it is done with the counting pass.
template <int NT, int ROWS, int LOG_NB, typename SH, typename Pad, typename Counted>
__device__ __forceinline__ GatherResult hinted_gather(SH& sh, const float (&v)[ROWS][4], Pad set_padding, Counted counted,
                                                      uint32_t hint_lo, uint32_t hint_hi, float mad_hint,
                                                      uint32_t k0, uint32_t k1, uint32_t* umax_slot) {
    GatherResult out = {PLAN_NONE, 0u, 0u};
    constexpr int NB = 1 << LOG_NB;
    const uint32_t span0 = hint_hi - hint_lo;
    const int shift = shift_for<LOG_NB>(span0);
    // the bracket (`bracket_counts` has let it pass) is widened to all NB buckets, less than twice the
    // hint's span, and starts on a bucket boundary
    const uint32_t lo = hint_lo & ~((1u << shift) - 1u);
    uint32_t* const cnt = sh.dlo;                  // 64 + NB + 64 counters
    // ---- pass 1: count
    {
        const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1);
        const BracketCounters<LOG_NB> counters(lo >> shift, lane);
        const uint32_t kb = opaque_s(counters.base);
        const uint32_t sh_s = opaque_s((uint32_t)shift);
        uint32_t um = 0;
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            float(&row)[4] = const_cast<float(&)[4]>(v[j]);
            asm volatile("" : "+v"(row[0]), "+v"(row[1]), "+v"(row[2]), "+v"(row[3]));
            um = max(max(um, __float_as_uint(row[0])), __float_as_uint(row[1]));
            um = max(max(um, __float_as_uint(row[2])), __float_as_uint(row[3]));
            set_padding(j);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t at = counters.at(__float_as_uint(row[i]) >> sh_s, kb, [](float x, float l, float h) { return __builtin_amdgcn_fmed3f(x, l, h); });
                atomicAdd(reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(cnt) + at), 1u);
            }
            asm volatile("" : "+v"(um));
            __builtin_amdgcn_sched_barrier(0);
        }
        um = wave_max_to_last(um);
        if (lane == WAVE - 1) atomicMax(umax_slot, um);
    }
    // Waves of other workgroups of the CU may be anywhere in their columns: the short phases, whose
    // length is a chain of latencies, go before the counting pass (bound by LDS), that before the
    // gathers and these before the scores, which are bound by issue (launch: 32 768 ranks x 4 096 x 8
    // 1 027 us with no priorities, 990 with the short phases' alone, 976 so; 16 384 x 10 000 x 4 741, 724, 721).
    __builtin_amdgcn_s_setprio(3);
    counted();
    __syncthreads();
    const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1), w = rfl(tid >> 6);
    const uint32_t umax = rfl(*umax_slot);
    out.umax = umax;
    uint32_t top = umax;                   // (of the samples that arrived)
    if (__builtin_expect(umax > 0x7F800000u && umax < 0x80000000u, 0)) {
        // missing samples (NaNs): counted over the bracket like any large value, they only
        // move the ranks asked for
        count_present(sh, v, &out.present, &top);
        k0 = out.present ? (out.present - 1) / 2 : 0u;
        k1 = out.present / 2;
    }
    // the lane-private words: everything under the bracket is `below`
    if (w == 0) {
        uint32_t d = cnt[lane];
        cnt[lane] = 0;
        d = wave_incl_scan(d);
        if (lane == WAVE - 1) sh.below = d;
    }
    if (w == 1u) cnt[64 + NB + lane] = 0;
    uint32_t below;
    const bool bracketed = locate<NT, LOG_NB, true, true>(sh, tid, k0, k1, &below);
    if (top > BRACKET_KEY_LIMIT || !bracketed) return out;
    if (w == 0) plan_gather<LOG_NB>(sh, lane, lo, shift, mad_hint, below, k0, k1);
    __syncthreads();
    // (all of it at once: read where it is used it is a chain of LDS latencies)
    const GatherPlan plan = sh.plan;
    const float center = uniform(plan.center), inner = uniform(plan.inner), reach = uniform(plan.reach);
    const uint32_t wspan = rfl(__float_as_uint(plan.outer - plan.inner));
    const uint32_t lb0 = rfl(plan.lb0), lspan = rfl(plan.li - plan.lb0), rb0 = rfl(plan.rb0), rspan = rfl(plan.rx - plan.rb0);
    const uint32_t mid_p = rfl(plan.mid), ba = mid_p & 0xFFFFu, cspan = mid_p >> 16, n_dist = rfl(plan.n_out - plan.n_in);
    out.status = rfl(plan.status);
    if (out.status == PLAN_GATHER && n_dist > MOST_DIST) out.status = PLAN_LOCATED;
    out.umax = out.status == PLAN_NONE ? umax : top;
    if (__builtin_expect(out.status != PLAN_GATHER, 0)) return out;
    // ---- gather the rows that hold a value of the median's buckets or of the MAD's
    // (128 rows of a wave where the counters have room for them, up to 512 threads: a sample's wide
    // bracket has up to twice the candidates, and with 64 rows one in twenty first columns of 16 384
    // ranks overflowed a list of one of its four waves)
    RowList<SH, SH::NB / (4 * SH::WAVES) < 128 ? 64 : 128> rows(sh, w);
    {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const float c = uniform(center), e = uniform(inner);
            float y[4];
            uint32_t off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                y[i] = v[j][i] - c;
                off[i] = __float_as_uint(fabsf(y[i]) - e);           // (negative: a large pattern)
            }
            const float near = fminf(fminf(fabsf(y[0]), fabsf(y[1])), fminf(fabsf(y[2]), fabsf(y[3])));
            const uint32_t far = min(min(off[0], off[1]), min(off[2], off[3]));
            rows.add(near <= reach || far <= wspan, v[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(3);
        rows.drain(lane, [&](uint32_t x, bool valid) {
            // (values under the bracket wrap round: (x - lo) >> shift is beyond every bucket)
            const uint32_t b = (x - lo) >> shift;
            const bool mid = valid && b - ba <= cspan, dist = valid && (b - lb0 < lspan || b - rb0 < rspan);
            const uint64_t mids = gd_ballot(mid), dists = gd_ballot(dist);
            if ((mids | dists) == 0ull) return;
            uint32_t base = 0;            // both counts in one word
            if (lane == 0) base = atomicAdd(&sh.ncand, (uint32_t)__popcll(mids) << 16 | (uint32_t)__popcll(dists));
            base = rfl(base);
            const uint64_t of = mid ? mids : dists;
            const uint32_t to = __builtin_amdgcn_mbcnt_hi((uint32_t)(of >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)of, mid ? base >> 16 : base & 0xFFFFu));
            // (the median's as keys of their own each: the offset in their buckets, then the place)
            if (mid && to < MOST_MID) sh.cand[to] = (x - (lo + (ba << shift))) << 6 | to;
            if (dist && to < MOST_DIST) sh.cand[MOST_MID + to] = x;
        });
    }
    __syncthreads();
    return out;
}

// The rest of the hinted selection where the gathered candidates did not settle it, or would have
// been too many: the median's bucket(s), located by hinted_gather, first, and then the MAD's.
template <int NT, int ROWS, int LOG_NB, typename SH>
__device__ __forceinline__ HintedResult hinted_rest(SH& sh, const float (&v)[ROWS][4], float mad_hint, uint32_t k0, uint32_t k1) {
    HintedResult out = {1, 0u, 0u, 0u, 0u, 0u};
    constexpr int NB = 1 << LOG_NB;
    constexpr uint32_t bmax = (uint32_t)NB - 1u;
    const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1), w = rfl(tid >> 6);
    const uint32_t lo = rfl(sh.plan.lo);
    const int shift = (int)rfl(sh.plan.shift);
    const uint32_t hi = lo + ((uint32_t)NB << shift) - 1u;
    const uint32_t ba = rfl(sh.res[0]), pa = rfl(sh.res[1]);
    const uint32_t bb = rfl(sh.res[2]), pb = rfl(sh.res[3]), below = rfl(sh.plan.skip) - pa;
    // ---- pass 2: the median's bucket(s)
    RowList<SH> rows(sh, w);
    {
        const uint32_t clo = lo + (ba << shift);
        const uint32_t cspan = ((bb - ba + 1u) << shift) - 1u;
        const uint32_t tok = opaque_s(clo);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            uint32_t off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) off[i] = __float_as_uint(v[j][i]) - tok;
            rows.add(min(min(off[0], off[1]), min(off[2], off[3])) <= cspan, v[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(3);
        rows.drain(lane, [&](uint32_t x, bool valid) {
            const bool hit = valid && x - tok <= cspan;
            append(lane, sh.cand, &sh.ncand, hit, x);
        });
    }
    __syncthreads();
    if (__builtin_expect(rfl(sh.ncand) != pb - pa, 0))           // (a wave's list was too short)
        gather_singly<ROWS>(sh, XKeys<ROWS, true>{v}, lo + (ba << shift), ((bb - ba + 1u) << shift) - 1u);
    rank_candidates<NT>(sh, tid, pb - pa, k0 - below - pa, k1 - below - pa);
    if (tid == 0) sh.ncand = 0;
    const uint32_t s0 = rfl(sh.res[4]), s1 = rfl(sh.res[5]);
    out.m0 = s0; out.m1 = s1;
    const float med = 0.5f * (__uint_as_float(s0) + __uint_as_float(s1));
    if (!(mad_hint > 0.0f)) return out;
    // ---- MAD: search the prefix sums.  Candidate e is a right edge (a bucket's lower
    // edge, e > bb); its distance from the median mirrored to the left gives the edge
    // f, the first one above the mirror point.  F = #[f, e) never decreases with e.  Every wave
    // looks at 64 edges around the one that the hint points at, one a lane, for itself: no barrier.
    // Should they not hold the answer, it looks at every sixteenth of the 1 024 about them and then
    // at the 64 where those point (a hint that is 17 % off, one step: 16 384 ranks x 4 16.0 -> 15.0 us,
    // 5 000 x 2 14.6 -> 13.7 against steps of 32 edges at a time).
    auto edge = [&](uint32_t e) { return __uint_as_float(lo + (e << shift)); };
    const uint32_t kr = __float_as_uint(med + mad_hint);
    uint32_t e0 = (kr >= lo && kr <= hi ? (kr - lo) >> shift : bmax) - 32u;     // the first lane's edge (mod 2^32)
    uint32_t Rb0 = 0, Rb1 = 0, Lb0 = 0, Lb1 = 0;
    bool found = false;
    uint32_t step = 1;
    for (int round = 0; round < 3; ++round) {
        const uint32_t e = e0 + lane * step;
        uint32_t f = 0, F = 0;
        bool valid = e > bb && e <= bmax + 1u;                    // (wraps below 0: beyond bmax)
        if (valid) {
            const float d = edge(e) - med;
            const uint32_t kl = __float_as_uint(med - d);
            f = ((kl - lo) >> shift) + 1u;
            valid = d > 0.0f && kl >= lo && kl <= hi && f <= e;
            if (valid) F = sh.pref[e] - sh.pref[f];
        }
        const uint64_t under = gd_ballot(valid && F <= k0), over = gd_ballot(valid && F > k1);
        if (round == 1) {                                          // the fine look, about where the coarse one points
            if (over == 0ull || under == 0ull) break;
            e0 += 16u * (63u - (uint32_t)__builtin_clzll(under)) - 24u;
            step = 1;
            continue;
        }
        if (over == 0ull || under == 0ull) {                       // not here: every sixteenth edge, 512 to either side
            e0 -= 32u * 15u;
            step = 16;
            continue;
        }
        // The last edge with at most k0 values inside: at most as many are closer than f, the edge
        // that it gives on the left.  Buckets grow wider with their values, so that f's own mirror
        // image lies in the bucket before the right edge.  (A bucket further in on both sides has
        // twice as many distances to rank where the left ones are narrow: exponential values, 56 000
        // ranks x 1 024 143 us, so 112.)
        const uint32_t la = 63u - (uint32_t)__builtin_clzll(under), lb = (uint32_t)__builtin_ctzll(over);
        Rb0 = rfl(e0 + la - 1u);
        Rb1 = rfl(e0 + lb - 1u);
        Lb1 = (uint32_t)__builtin_amdgcn_readlane((int)f, (int)la) - 1u;
        Lb0 = (uint32_t)__builtin_amdgcn_readlane((int)f, (int)lb) - 1u;
        found = true;
        break;
    }
    // Bucket ranges: the distances wanted end in the buckets Rb0..Rb1 on the right of the
    // median, Lb0..Lb1 on its left.
    if (!found || Rb0 <= bb || Rb1 > bmax || Rb0 > Rb1 || Lb1 >= ba || Lb0 > Lb1) return out;
    const float dLi = med - edge(Lb1 + 1u), dLo = med - edge(Lb0);
    const float dRi = edge(Rb0) - med, dRo = edge(Rb1 + 1u) - med;
    const float DI = fmaxf(dLi, dRi), DO = fminf(dLo, dRo);
    const float Da = fminf(dLi, dRi), Db = fmaxf(dLo, dRo);
    const uint32_t n_in = rfl(sh.pref[Rb0] - sh.pref[Lb1 + 1u]);
    if (!(Da > 0.0f) || !(DO >= DI)) return out;
    // ---- pass 3: gather the rows that hold a value of these buckets, and classify their values exactly
    {
        const float tokm = __uint_as_float(opaque_s(__float_as_uint(med)));
        const float toka = __uint_as_float(opaque_s(__float_as_uint(Da)));
        const uint32_t wspan = __float_as_uint(Db - Da);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            uint32_t off[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) off[i] = __float_as_uint(fabsf(v[j][i] - tokm) - toka);   // negative: a large pattern
            rows.add(min(min(off[0], off[1]), min(off[2], off[3])) <= wspan, v[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(3);
        if (rows.overflow() && lane == 0) atomicAdd(&sh.nkept, (uint32_t)CAND_CAP + 1u);
        rows.drain(lane, [&](uint32_t x, bool valid) {
            // (values under the bracket wrap round: (x - lo) >> shift is beyond every bucket)
            const uint32_t b = (x - lo) >> shift;
            const bool in = valid && (b - Lb0 <= Lb1 - Lb0 || b - Rb0 <= Rb1 - Rb0);
            const float d = fabsf(__uint_as_float(x) - med);
            const uint32_t nlt = (uint32_t)__popcll(gd_ballot(in && d < DI));
            if (nlt != 0 && lane == 0) atomicAdd(&sh.nnear, nlt);
            append(lane, sh.cand, &sh.nkept, in && d >= DI && d <= DO, __float_as_uint(d));
        });
    }
    __syncthreads();
    const uint32_t c_in = n_in + rfl(sh.nnear), kept = rfl(sh.nkept);
    // Each candidate is compared with all: beyond a few hundred it is sooner to select among all the
    // distances.  Crowds of equal values about an edge, ranked / selected, 32 768 ranks x 1 024 x 2: 120
    // of them 102 / 104 us, 160 109 / 104, 400 165 / 116; 65 536 x 512 x 4: 160 183 / 195, 200 197 / 201,
    // 240 215 / 203, 400 322 / 212; 16 384 x 2 048 x 2: 80 99 / 109, 120 123 / 119, 200 147 / 140.
    constexpr uint32_t MOST_RANKED = NT >= 1024 ? 224 : 128;
    static_assert(MOST_RANKED <= (uint32_t)CAND_CAP, "the candidates fit their list");
    const bool ok = kept <= MOST_RANKED && c_in <= k0 && k1 < c_in + kept;
    out.q0 = k0 - c_in; out.q1 = k1 - c_in;
    out.listed = kept;
    if (__builtin_expect(!ok || kept > (uint32_t)WAVE, 0)) {
        if (ok) {
            rank_candidates<NT>(sh, tid, kept, k0 - c_in, k1 - c_in);
            out.q0 = rfl(sh.res[4]);
            out.q1 = rfl(sh.res[5]);
            out.listed = 0;
        } else {
            __syncthreads();
        }
        if (tid == 0) {          // (a zero made here: kept in registers for the whole kernel it ends up spilled)
            const uint32_t zero = opaque_v(0u);
            sh.nkept = zero; sh.nnear = zero;
        }
        if (!ok) return out;
    }
    out.found = 2;
    return out;
}

// Hints for columns that have no predecessor to take them from (the first step of a workgroup's
// run): median and quartiles of a sample.  Like all hints they are only trusted as far as the
// counting pass of the hinted selection confirms them, whatever the column holds.
// All columns of the step are sampled at once, ahead of everything else and while the first column
// is on its way: a wave takes 256 values of one column, sorts them as four lots of 64 by lane
// exchanges and averages the lots' quartiles; up to four waves share a column.  (A sample of every
// column in its turn, four values of every thread by way of a histogram, took five barriers and 4 000
// to 6 000 cycles a column: launch, 5 000 ranks x 1 000 x 2 29.2 us, so 26.4, 20 000 x 512 x 3 48 and 43, 40 000 x
// 256 x 8 102 and 92.5, x 1 024 336 and 326, 65 536 x 512 x 8 279 and 258, x 4 096 1 836 and 1 815, 32 768 x 512 x 8
// with z 224 and 216.)

// Four lots of 64 keys, into ascending order each: a lane keeps the smaller or the larger key of a
// stage by way of the median of the two and of 0 or ~0.
template <int J, int S>
__device__ __forceinline__ void exchange_lots(uint32_t (&v)[4]) {
    const uint32_t bound = gd_lane_in<gd_keeps_smaller<J, S>(), true>() ? 0u : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t o;
        if constexpr (J == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(v[i], v[i], false, false);
            o = gd_lane_in<gd_lanes_with<16>(), true>() ? r[0] : r[1];
        } else if constexpr (J == 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(v[i], v[i], false, false);
            o = gd_lane_in<gd_lanes_with<32>(), true>() ? r[0] : r[1];
        } else {
            o = gd_lane_xor<J>(v[i], 0);
        }
        v[i] = max(min(v[i], o), min(max(v[i], o), bound));
    }
}
template <int S>
__device__ __forceinline__ void merge_lots(uint32_t (&v)[4]) {
    if constexpr (S > 32) exchange_lots<32, S>(v);
    if constexpr (S > 16) exchange_lots<16, S>(v);
    if constexpr (S > 8) exchange_lots<8, S>(v);
    if constexpr (S > 4) exchange_lots<4, S>(v);
    if constexpr (S > 2) exchange_lots<2, S>(v);
    exchange_lots<1, S>(v);
}

// Quartiles of a wave's 256 values (missing samples, NaNs, are left out): the middle one is a NaN
// where the sample says that hints would not hold -- signs, too few values, or few distinct ones (three
// alike in the middle of two lots or more), whose buckets the hinted selection would find crowded
// and give up after its counting pass.  (Whole degrees, 65 536 ranks x 256 x 4 385 us where an eighth of
// a lot had to be alike, so 308, 8 000 x 1 000 x 4 249 and 205.  The MAD comes of the quartiles, see
// mad_of_quartiles: by the lots' own distances plain columns took longer, 12 000 x 1 000 x 4 56.0 and
// 57.7, and values in two heaps, 5 000 x 1 000 x 2 35 and 52.)
__device__ __forceinline__ void sample_quartiles(uint32_t (&k)[4], float* q25, float* q50, float* q75) {
    uint32_t top = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) top = max(top, k[i]);
    const bool signs = gd_ballot(top >= 0x80000000u) != 0ull;
    merge_lots<2>(k); merge_lots<4>(k); merge_lots<8>(k);
    merge_lots<16>(k); merge_lots<32>(k); merge_lots<64>(k);
    float s25 = 0.0f, s50 = 0.0f, s75 = 0.0f;
    uint32_t lots = 0, alike = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t n = (uint32_t)__popcll(gd_ballot(k[i] <= 0x7F800000u));
        auto at = [&](uint32_t rank) { return (uint32_t)__builtin_amdgcn_readlane((int)k[i], (int)(rank & (WAVE - 1))); };
        if (n >= 16u) {
            s25 += __uint_as_float(at(n / 4)); s50 += __uint_as_float(at(n / 2)); s75 += __uint_as_float(at(n - 1u - n / 4));
            alike += at(n / 2 - 1u) == at(n / 2 + 1u) ? 1u : 0u;
            ++lots;
        }
    }
    const float share = lots == 4u ? 0.25f : lots == 3u ? 1.0f / 3.0f : lots == 2u ? 0.5f : 1.0f;
    const bool none = signs || lots == 0u || alike >= 2u;
    *q25 = s25 * share;
    *q50 = none ? __uint_as_float(0x7FC00000u) : s50 * share;
    *q75 = s75 * share;
}

// The MAD of a sample whose quartiles lie `left` and `right` of its median, `half` their mean: that, and
// less of it where one side is the wider one.  Of exponential, log-normal and gamma distributed values it
// is `half` times the fourth power of the sides' geometric mean over `half`, to 3 %; where that would be
// less than a half of it, the column is no skewed heap but several.  (`half` alone, launch, exponential
// values / log-normal ones of sigma 1: sampled all at once, with a reach that then went below zero and
// left the column without hints, 8 000 ranks x 1 000 x 4 90 / 88 us, so 50 / 49, 12 000 x 1 000 x 4 105 / 104 and
// 62 / 63, 32 768 x 512 x 8 209 / 203 and 126 / 126; one by one, 16 384 x 1 024 x 4 115 / 95 and 73 / 75, 4 096 x 256 x 1
// 20.3 / 19.6 and 12.2 / 12.2, one step of 20 000 x 4 21.4 / 17.6 and 17.1 / 17.2.  Even columns and such in two
// heaps the same within 1 %.)
__device__ __forceinline__ float mad_of_quartiles(float left, float right, float half) {
    const float per = __builtin_amdgcn_rcpf(half), even = (left * per) * (right * per), share = even * even;
    return share >= 0.5f ? half * share : half;
}

// The same for a column whose first register row has come: a sample of four values of every thread (row 0, which covers the whole
// rank range), its median and quartiles read off a histogram over the sample's own range (one step
// of 20 000 ranks x 4, no hints: 17.0 us; 18.2 by sorted lots).  Thread 0 writes the hints of metric m;
// ends with a barrier, the work area at rest.  (missing samples are left out)
template <int NT, int LOG_NB, typename SH>
__device__ __forceinline__ void sample_hints(SH& sh, const float (&row)[4], uint32_t m) {
    constexpr int BPT = (1 << LOG_NB) / NT;
    const uint32_t tid = opaque_v(threadIdx.x), lane = tid & (WAVE - 1);
    uint32_t k[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) k[i] = __float_as_uint(row[i]);
    uint32_t mn = 0xFFFFFFFFu, mx = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool in = (k[i] & 0x7FFFFFFFu) <= 0x7F800000u;
        mn = in ? min(mn, k[i]) : mn;
        mx = in ? max(mx, k[i]) : mx;
    }
    mn = wave_min_to_last(mn);
    mx = wave_max_to_last(mx);
    if (lane == WAVE - 1) { atomicMin(&sh.smin, mn); atomicMax(&sh.smax, mx); }
    __syncthreads();
    const uint32_t smin = rfl(sh.smin), smax = rfl(sh.smax);
    const int sshift = shift_for<LOG_NB>(smax - smin);
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if ((k[i] & 0x7FFFFFFFu) <= 0x7F800000u) atomicAdd(&sh.hist[(k[i] - smin) >> sshift], 1u);
    __syncthreads();
    if (tid == 0) { sh.smin = 0xFFFFFFFFu; sh.smax = 0; }
    uint32_t loc[BPT], sum = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) { loc[q] = sh.hist[tid * BPT + q]; sum += loc[q]; }
#pragma unroll
    for (int q = 0; q < BPT; ++q) sh.hist[tid * BPT + q] = 0;
    uint32_t n;
    const uint32_t excl = block_excl_scan<NT>(sum, tid, sh.wpart, &n);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const uint32_t want = (uint32_t)(r + 1) * (n / 4) - excl;      // sample ranks n/4, n/2, 3n/4
        if (want < sum) {
            uint32_t p = 0;
            bool done = false;
#pragma unroll
            for (int q = 0; q < BPT; ++q) {
                if (!done && want - p < loc[q]) {
                    sh.res[r] = r == 1 && loc[q] > n / 8 ? 0xFFFFFFFFu : tid * BPT + q;
                    done = true;
                }
                p += loc[q];
            }
        }
    }
    __syncthreads();
    // (more than an eighth of the sample in the middle's bucket: few distinct values, whose buckets
    // the hinted selection would find crowded and give up after its counting pass)
    if (tid == 0 && n != 0 && sh.res[1] != 0xFFFFFFFFu) {
        const uint32_t half = (1u << sshift) >> 1;
        const float q25 = __uint_as_float(smin + (sh.res[0] << sshift) + half);
        const float q50 = __uint_as_float(smin + (sh.res[1] << sshift) + half);
        const float q75 = __uint_as_float(smin + (sh.res[2] << sshift) + half);
        const float sides = 0.5f * (q75 - q25), hd = mad_of_quartiles(q50 - q25, q75 - q50, sides);
        if (q50 > 0.0f && hd > 0.0f && q50 < 3.0e38f && hd < 3.0e38f) {      // (false for NaNs)
            sh.hmed[m] = q50;
            // (the reach a run keeps from step to step, on the left no further than half way from where the MAD ends to zero)
            sh.hwl[m] = fminf(1.25f * sides, 0.5f * (q50 + hd));
            sh.hwh[m] = 1.25f * sides;
            sh.hmad[m] = hd;
            sh.hok[m] = 1;
        }
    }
    __syncthreads();
}

// The signs of four words, byte by byte in order: those bits of `bits` are set whose byte's word is
// negative.  (A permute's selectors 9 and 11 fill a byte with the sign of a word, so that what
// remains is one operation of three inputs; with the words' top bytes brought together, shifted
// and masked it was five instructions a row instead of three: launch, 5 000 ranks x 10 000 x 2 157 us,
// so 155, 65 536 x 4 096 x 8 1 839 and 1 835.)
__device__ __forceinline__ uint32_t sign_bytes(uint32_t d0, uint32_t d1, uint32_t d2, uint32_t d3, uint32_t bits) {
    const uint32_t lo2 = __builtin_amdgcn_perm(d1, d0, 0x0C0C0B09u);
    const uint32_t hi2 = __builtin_amdgcn_perm(d3, d2, 0x0B090C0Cu);
    return (lo2 | hi2) & bits;
}

// Signed score and node score of one register row, dividing with the IEEE
// operator.  agg 0 = scaled pairwise sum, 1 = max (uniform).  This is the route of every
// column that holds a missing sample.
__device__ __forceinline__ void score_row(uint32_t agg, const float (&x)[4], float med, float s, uint32_t absmask,
                                          uint32_t sgnmask, float thr, float node_scale,
                                          uint32_t* e, float* nz) {
    float zs[4];
    uint32_t bits = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float z = ((x[i] + 0.0f) - med) / s;      // -0 reads as +0
        const float zi = __uint_as_float((__float_as_uint(z) & absmask) ^ sgnmask);
        // A NaN is a missing sample and its score a NaN: it never exceeds (the
        // comparison is false) and adds nothing to its node.
        bits |= (zi > thr ? 1u : 0u) << (8 * i);
        zs[i] = zi == zi ? zi : 0.0f;
    }
    *e = bits;
    // lanes 2p and 2p+1 hold GPUs 0-3 and 4-7 of one node
    if (agg == 0) {
        const float half = (zs[0] + zs[1]) + (zs[2] + zs[3]);
        const float other = lane_xor1(half);
        *nz = node_scale * (half + other);
    } else {
        const float half = fmaxf(fmaxf(zs[0], zs[1]), fmaxf(zs[2], zs[3]));
        const float other = lane_xor1(half);
        *nz = fmaxf(half, other) + 0.0f;
    }
}

// The same for the scaled sum, with the quotient d/s obtained from the
// column's reciprocal r = RN(1/s) by two residual corrections:
//   q0 = RN(d*r); q1 = RN(q0 + RN(d - q0*s)*r); q2 = RN(q1 + (d - q1*s)*r)
// q1 is within one ulp of d/s, for which the residual d - q1*s is exact in
// fp32 and the second correction returns the correctly rounded quotient
// (Markstein's division theorem), provided nothing under- or overflows --
// the caller checks the column's magnitudes for that.  ss is +s or -s (a
// lower-is-worse metric scores -z), TWO_SIDED scores |z|.
// The exceed bits are those of `bits` (one in each byte).
template <bool TWO_SIDED>
__device__ __forceinline__ void score_row_fast(const float (&x)[4], float med, float ss, float rs, float thr,
                                               float node_scale, uint32_t bits, uint32_t* e, float* nz) {
    float zs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float d = x[i] - med;
        const float q0 = d * rs;
        const float e0 = __builtin_fmaf(-q0, ss, d);
        const float q1 = __builtin_fmaf(e0, rs, q0);
        const float e1 = __builtin_fmaf(-q1, ss, d);
        const float q2 = __builtin_fmaf(e1, rs, q1);
        zs[i] = TWO_SIDED ? fabsf(q2) : q2;
    }
    // (finite numbers and a threshold that is not -0, which less a score of +0 would be negative: a
    // score exceeds iff thr less it is negative, denormals being kept.  Compared value by value / so,
    // 1 024 steps x 8: two-sided metrics 40 000 ranks 386 / 382 us, 65 536 541 / 539; one-sided ones,
    // of which only the primary comes here, the same within 0.5 %)
    *e = sign_bytes(__float_as_uint(thr - zs[0]), __float_as_uint(thr - zs[1]), __float_as_uint(thr - zs[2]),
                    __float_as_uint(thr - zs[3]), bits);
    const float half = (zs[0] + zs[1]) + (zs[2] + zs[3]);
    const float other = lane_xor1(half);
    *nz = node_scale * (half + other);
}

// Supporting (non-primary) metric with a one-sided direction, sign-free column:
// only the decisions are needed, not the scores, so no division is done.
//   * A rank exceeds iff x >= xstar (higher is worse) or x <= xstar (lower is
//     worse): sub and divide are monotone, and xstar is the exact boundary found
//     with the very operations the definition uses.
//   * The node score scale*sum(z') is estimated as cc*sum(x) - kk with
//     cc ~ +-scale/s and kk ~ 8*med*cc.  All roundings of the exact chain and of
//     the estimate together stay below `margin` (see the caller), so the estimate
//     decides unless it falls within `margin` of the threshold.  The estimate is
//     monotone in sum(x), so that a bound on the sum itself, checked against the
//     estimate's own formula where it is worked out (work_out), passes over the rows
//     in which no node exceeds or comes near.  In the others the estimate is formed
//     and, within `margin` of the threshold, the exact score.
//
// Values, sums and their bounds are not negative, and such floats order like their bit patterns.
// Of the bound b, `flip` is all ones and `cut` is b where higher is worse, `flip` is 0 and `cut` is
// ~b where lower is: the sign of (x ^ flip) + cut, b - 1 - x or x - b - 1, is the decision, in one
// instruction and the same code for both directions.
__device__ __forceinline__ uint32_t decided(float x, uint32_t flip, uint32_t cut) {
    return (__float_as_uint(x) ^ flip) + cut;
}

// FULL: R == NT*4*ROWS exactly, so no lane is padding and no bounds are checked.  A ragged
// rank count takes a tiling of at most two rows too many (NT*4*(ROWS-2) < R): only the
// last two rows can hold padding lanes and only they are checked, at compile time, so that
// they take the hinted selection at the cost of an exact fit.  Measured (launch): 40 000
// ranks x 1 024 steps x 8 metrics 571 us with one tiling up to the next power of two, every
// row checked and the general selection, 585 us with empty rows passed over at run time
// (scalars spilled and registers copied at every check), 403 us this way; 5 000 x 1 000 x 2
// 60 -> 45 us; 65 528 ranks take 600 us where 65 536 take 583.
// SPLIT (short batches, the streaming case): one workgroup per column instead of
// per run of steps, so that the M columns of a step are scored side by side.  The
// exceed bits of a column then go out as bit planes and combine_kernel makes the mask
// bytes of them and applies the multi-signal rule.
// The kernel's arguments, read from its argument segment where they are used: kept in scalar
// registers across the column loop they are most of what the compiler has to spill there.
typedef const __attribute__((address_space(4))) gd_score_args* gd_args_ptr;
__device__ __forceinline__ gd_args_ptr args_here() {
    gd_args_ptr p = (gd_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// Rows of the next column that the 1 024-thread tilings have registers to spare for (128 a lane).
// They are asked for as soon as the current column is counted: a workgroup has its CU to itself
// there, and from the count to the scores the memory has nothing to do.  Measured: ten rows, 40 000
// ranks x 1 024 steps x 8: none 399 us, three 391, five 383, six 382, seven 390; twelve, 48 000 x
// 2 048 x 4: none 471, two 471, three 465, four 460, five 456; fourteen, 56 000 x 2 048 x 4: none
// 532, two 538, three 532.  The six and the five hold over their whole tilings: 33 000, 36 000 and 40 952
// ranks x 1 024 steps x 8 without / with them 364 / 355, 364 / 353 and 389 / 368 us, 41 000, 44 000 and 49 144
// 415 / 393, 419 / 399 and 444 / 417 (2 048 x 4 and 1 500 x 2: 3 to 7 %).  With fewer threads other
// workgroups of the CU fill the gap (up to eight rows kept this way: 5 000 to 24 000 ranks within 1 %).
constexpr int rows_ahead(int nt, int rows) {
    return nt < 1024 ? 0 : rows == 10 ? 6 : rows == 12 ? 5 : 0;
}

template <int NT, int ROWS, int LOG_NB, bool FULL, bool SPLIT, bool WANT_Z>
__device__ __forceinline__ void score_columns(const gd_score_args& a) {
    constexpr int TAIL = FULL ? ROWS : (ROWS > 2 ? ROWS - 2 : 0);     // first row that may hold padding
    constexpr int BLK = NT * 4;               // ranks per register row
    constexpr int MAX_NODES = BLK * ROWS / 8;
    constexpr int NWAVES = NT / WAVE;
    // Where the first step's columns are sampled all at once (see sample_quartiles), and where one by
    // one: with one column in a workgroup, and in the exact fits of 256 threads and in sixteen rows of them, of
    // which plain columns in runs of one step gain by the larger sample (one by one / all at once, launch:
    // 4 096 x 256 x 1 11.6 / 12.0 us, 15 000 x 1 024 x 4 70.2 / 73.4, 16 384 x 1 024 x 4 70.9 / 71.4; fewer rows,
    // 12 000 x 1 000 x 4 61.5 / 56.2).  Longer runs gain nothing either way (15 000 x 3 000 x 4 194 / 194, 16 384 x
    // 10 000 x 4 605 / 606), more metrics would lose (16 384 x 512 x 8 94.0 / 90.5), and so do columns in two heaps or of
    // few distinct values, which the lots find out sooner (16 384 x 1 024 x 4 110 / 82 and 406 / 333).  (A batch's
    // ragged tiling of up to four rows is through the general route sooner: 4 000 ranks x 256 steps, one
    // metric, 16.7 us that way, 19.5 with a sample's hints.)
    constexpr bool SAMPLES = !SPLIT && (NT > 256 || (!FULL && ROWS > 4 && ROWS < 16));
    constexpr bool SAMPLES_SINGLY = SPLIT || (NT <= 256 && (FULL || ROWS == 16));
    using SH = Shared<NT, LOG_NB, MAX_NODES>;
    // Dynamic LDS: the selection's work area, then one word of exceed-mask bytes
    // per (row, thread) -- kept in LDS, not registers, across the M columns.
    extern __shared__ __align__(16) unsigned char lds_raw[];
    SH& sh = *reinterpret_cast<SH*>(lds_raw);
    uint32_t* emask = reinterpret_cast<uint32_t*>(lds_raw + ((sizeof(SH) + 15) & ~(size_t)15));

    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int w = rfl(tid >> 6);
    // (opaque: four words of a tuple otherwise, which is spilled as a whole)
    const uint32_t R = opaque_s(a.R), N = opaque_s(a.N), M = opaque_s(a.M);
    const uint32_t RW = (R + 63) / 64, NWD = (N + 63) / 64;
    // Each workgroup scores a contiguous run of steps, column after column, and
    // loads the next column while it scores the current one.
    const uint32_t spw = SPLIT ? 1u : (a.T + gridDim.x - 1) / gridDim.x;
    const uint32_t t_begin = SPLIT ? blockIdx.x / M : blockIdx.x * spw;
    const uint32_t t_end = min(a.T, t_begin + spw);
    if (t_begin >= t_end) return;
    const uint32_t m_begin = SPLIT ? blockIdx.x % M : 0u, m_end = SPLIT ? m_begin + 1u : M;

    // Row j of wave w covers rank block (j + w) % ROWS, so that the first
    // registers to arrive (row 0) sample the whole rank range.  (The rows that may hold
    // padding stay where they are.)
    // The lane part (tid*4) is passed in so that each phase can use its own,
    // optimiser-opaque copy: otherwise every row's store and load address is
    // computed once and kept in registers for the whole kernel.
    const int wrow = FULL ? w : (TAIL > 0 ? w % (TAIL > 0 ? TAIL : 1) : 0);
    auto block_of = [&](int j) -> uint32_t {
        if (FULL) return (uint32_t)((j + wrow) & (ROWS - 1));
        if (j >= TAIL) return (uint32_t)j;
        return (uint32_t)(j + wrow >= TAIL ? j + wrow - TAIL : j + wrow);
    };
    auto rbase = [&](int j, uint32_t tid4) -> uint32_t { return block_of(j) * BLK + tid4; };
    auto holds = [&](int j, uint32_t tid4) -> bool { return j < TAIL || rbase(j, tid4) < R; };
    auto fresh_tid4 = [&]() -> uint32_t { return opaque_v((uint32_t)tid * 4); };

    // The first step's samples (see sample_quartiles): wave w takes part w mod 2^SL of column w >> SL, or,
    // with fewer waves than columns, columns w, w + NWAVES, ..., and asks for them ahead of the first
    // column.
    constexpr int LOTS = (8 + NWAVES - 1) / NWAVES;
    const uint32_t columns = m_end - m_begin;
    const bool crowded = LOTS > 1 && columns > (uint32_t)NWAVES;
    const uint32_t sl = sample_parts_log(columns, NWAVES);
    auto column_of = [&](int p) -> uint32_t { return crowded ? (uint32_t)(w + p * NWAVES) : p == 0 ? (uint32_t)w >> sl : columns; };
    uint32_t lot[LOTS][4];
    if (SAMPLES) {
        const uint32_t from = sample_rank(((uint32_t)w & ((1u << sl) - 1u)) * WAVE + (uint32_t)lane, R);
#pragma unroll
        for (int p = 0; p < LOTS; ++p) {
            const float* col = a.x + ((size_t)t_begin * M + min(column_of(p), columns - 1u)) * R;
            const uint4 q = *reinterpret_cast<const uint4*>(col + from);
            lot[p][0] = q.x; lot[p][1] = q.y; lot[p][2] = q.z; lot[p][3] = q.w;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // Rows of the next column that the score loop asks for as it is done with each; the others
    // follow behind the loop.  Asked for row by row to the end, the loads fill the memory
    // pipeline and the loop's last rows wait for room in it (launch, 65 536 ranks x 4 096 x 8:
    // 2 115 us all in the loop, 2 081 with a quarter behind it, 2 045 half, 2 085 three quarters;
    // asked for by the next column's count, which is bound by LDS, 2 033, but then a column that
    // takes the general way waits for half of its values).
    constexpr int EARLY = SPLIT || rows_ahead(NT, ROWS) > 0 ? ROWS : (ROWS + 1) / 2;
    constexpr int AHEAD = SPLIT ? 0 : rows_ahead(NT, ROWS);
    float v[ROWS][4], ahead[AHEAD > 0 ? AHEAD : 1][4];
    // Issue the loads of one register row of a column.  Padding lanes read the column's last
    // ranks once more (a load under a condition would be waited for on the spot) and become
    // NaNs, whose key lies above every real key, when the column is first looked at.
    auto load_row_to = [&](float (&row)[4], int j, const float* col, uint32_t tid4) {
        // (a buffer's base, a scalar and the lane's 32-bit offset: one address mode, no vector arithmetic
        // per row; of a column, whose bytes bound it)
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(col), 0, (int)(R * 4u), 0x00020000);
        const int from = j < TAIL ? (int)(block_of(j) * BLK * 4u) : 0;
        const int lane_at = (int)(j < TAIL ? tid4 * 4u : min((uint32_t)j * BLK + tid4, R - 4) * 4u);
        // (a single step, just arrived, may still lie in the caches)
        const gd_u4 q = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_at, from, SPLIT ? 0 : NONTEMPORAL);
#pragma unroll
        for (int i = 0; i < 4; ++i) row[i] = __uint_as_float(q[i]);
    };
    auto load_row = [&](int j, const float* col, uint32_t tid4) { load_row_to(v[j], j, col, tid4); };
    auto load_ahead = [&](const float* col) {
        if (AHEAD == 0) return;
        const uint32_t ta = fresh_tid4();
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) load_row_to(ahead[j], j, col, ta);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto set_padding = [&](int j, uint32_t tid4) {
        if (j < TAIL) return;
        const bool pad = (uint32_t)j * BLK + tid4 >= R;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[j][i] = pad ? __uint_as_float(0x7FFFFFFFu) : v[j][i];
    };
    auto load_first = [&]() {
        const uint32_t tl = fresh_tid4();
        const float* col = a.x + ((size_t)t_begin * M + m_begin) * R;
        // issued in row order, like the refills of the score loop: the waits of the
        // first pass over a column are then placed row by row
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            load_row(j, col, tl);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (!SPLIT) load_first();

    uint32_t NE[(ROWS + 3) / 4]; // node mask byte per row, packed
    // the selection's work area starts in its rest state (see the LDS protocol)
    for (int i = tid; i < SH::NB + 128; i += NT) sh.dlo[i] = 0;      // dlo, hist, dhi
    for (int i = tid; i < (MAX_NODES / 8 > 0 ? MAX_NODES / 8 : 1); i += NT) sh.ranka[i] = 0;
    for (int i = tid; i < (int)CAND_REST; i += NT) sh.cand[i] = CAND_NONE;
    if (tid == 0) {
        sh.umax[0] = 0; sh.umax[1] = 0; sh.ncand = 0; sh.below = 0; sh.nkept = 0; sh.nnear = 0;
        sh.smin = 0xFFFFFFFFu; sh.smax = 0; sh.d1 = 0; sh.d2 = 0xFFFFFFFFu;
        for (int m = 0; m < 8; ++m) { sh.hok[m] = 0; sh.hfast[m] = 1; }
        // (the reciprocal is only used where node_scale > 0)
        sh.rules = {a.thr, a.node_scale, a.rel_floor, a.abs_floor, 1.0f / a.node_scale, a.node_agg};
        // A one-step call may be told the medians and MADs of a recent step (usually the
        // previous call's outputs).  They take the place of the hints a run of steps builds
        // up for itself; like those they are only trusted as far as the counting pass
        // confirms them, so any content is safe.
        if (SPLIT && a.hint_med && a.hint_mad && a.T == 1) {
            const float hm = a.hint_med[m_begin], hd = a.hint_mad[m_begin];
            if (hm > 0.0f && hd > 0.0f && hm < 3.0e38f && hd < 3.0e38f) {      // (false for NaNs)
                sh.hmed[m_begin] = hm;
                sh.hwl[m_begin] = 1.25f * hd;
                sh.hwh[m_begin] = 1.25f * hd;
                sh.hmad[m_begin] = hd;
                sh.hok[m_begin] = 1;
            }
        }
    }
    if (SAMPLES) {
        float* const found = reinterpret_cast<float*>(sh.pref);      // (not in use yet: three words a wave or column)
#pragma unroll
        for (int p = 0; p < LOTS; ++p) {
            const uint32_t c = column_of(p);
            if (c < columns) {
                float q25, q50, q75;
                sample_quartiles(lot[p], &q25, &q50, &q75);
                if (lane == 0) {
                    float* const to = found + 3u * (crowded ? c : (uint32_t)w);
                    to[0] = q25; to[1] = q50; to[2] = q75;
                }
            }
        }
    }
    __syncthreads();
    if (SPLIT) load_first();
    if (SAMPLES) {
        if ((uint32_t)tid < columns) {
            const float* const found = reinterpret_cast<const float*>(sh.pref) + 3u * ((uint32_t)tid << sl);
            float q25 = 0.0f, q50 = 0.0f, q75 = 0.0f;
            for (uint32_t i = 0; i < 1u << sl; ++i) { q25 += found[3 * i]; q50 += found[3 * i + 1]; q75 += found[3 * i + 2]; }
            const float share = 1.0f / (float)(1u << sl);
            const float mid = q50 * share, left = mid - q25 * share, right = q75 * share - mid, half = 0.5f * (left + right);
            const float hd = mad_of_quartiles(left, right, half);
            // the reach that a run keeps from step to step, and as much more as a small sample is off; on
            // the left no further than half way from where the MAD ends to zero
            const float reach = (sl >= 2u ? 1.25f : sl == 1u ? 1.375f : 1.5f) * half, low = fmaxf(mid - reach, 0.5f * (mid - hd));
            if (low > 0.0f && hd > 0.0f && mid < 3.0e38f && hd < 3.0e38f) {      // (false for NaNs)
                // The histogram covers up to twice what it must, above the bracket: half of the rest is
                // better below it.
                const uint32_t klo = __float_as_uint(low), span = __float_as_uint(mid + reach) - klo;
                const uint32_t rest = (1u << (LOG_NB + shift_for<LOG_NB>(span))) - span;
                const uint32_t c = m_begin + (uint32_t)tid;
                sh.hmed[c] = mid; sh.hmad[c] = hd;
                sh.hwl[c] = mid - __uint_as_float(klo - min(rest / 2u, klo));
                sh.hwh[c] = reach;
                sh.hok[c] = 1;
            }
        }
        __syncthreads();
    }
    constexpr uint32_t nsample = NT;          // (row 0, the column's sample, holds ranks throughout)
    uint32_t dir_codes = 0;          // direction + 1 of metric i in bits 2i, 2i + 1
#pragma unroll
    for (int i = 0; i < 8; ++i) dir_codes |= (uint32_t)(a.dir[i] + 1) << (2 * i);
    dir_codes = rfl(dir_codes);
    const uint32_t k0_all = R / 2 - 1, k1_all = R / 2;   // the middle ranks when nothing is missing (R is even)
    uint32_t colpar = 0;                          // parity of the column count: which umax slot is in use

    for (size_t t = t_begin; t < t_end; ++t) {
#pragma unroll
    for (int j = 0; j < ROWS; ++j) emask[j * NT + tid] = 0;   // each slot is private to its thread
#pragma unroll
    for (int j = 0; j < (ROWS + 3) / 4; ++j) NE[j] = 0;
    for (uint32_t m = m_begin; m < m_end; ++m) {
        // the column after this one (next metric, or the next step's first metric)
        // (after the very last column the current one is simply read again: a
        // branch-free refill keeps the register allocation of the score loops simple)
        const bool have_next = !SPLIT && (m + 1 < M || t + 1 < t_end);
        const float* this_col = args_here()->x + (t * M + m) * (size_t)R;
        const float* next_col = this_col + (have_next ? (size_t)R : 0);
        const uint32_t tl = fresh_tid4();
        // A workgroup scores consecutive steps, and telemetry moves little from one
        // step to the next: the previous step's median of this metric, with the
        // reach its histogram had, brackets this step's counting pass without
        // sampling.  A bracket that misses is noticed and replaced by the sample's.
        // (the first step of a run has no predecessor: a sample of the column stands in)
        bool boot = SAMPLES && t == t_begin;
        if (SAMPLES_SINGLY && t == t_begin && rfl(sh.hok[m]) == 0) {
            sample_hints<NT, LOG_NB>(sh, v[0], m);
            boot = true;
        }
        bool hinted = rfl(sh.hok[m]) != 0;
        uint32_t hint_lo = 0, hint_hi = 0;
        if (hinted) {
            const float xl = sh.hmed[m] - sh.hwl[m], xh = sh.hmed[m] + sh.hwh[m];
            hint_lo = rfl(__float_as_uint(xl));
            hint_hi = rfl(__float_as_uint(xh));
            hinted = xl >= 0.0f && xh > xl && hint_hi < 0x7F800000u;
        }
        uint32_t* const umax_slot = &sh.umax[colpar];
        // the other slot is free again: every thread read it a column ago
        if (tid == 0) sh.umax[colpar ^ 1u] = 0;
        colpar ^= 1u;
        uint32_t umax = 0;
        float med = 0.0f;
        uint32_t missing = 0;                   // the samples that arrived, where some did not
        bool special = false;                   // not scored by the fast routes: signs, or missing samples that stay
        // (all eight directions in one scalar word: indexing the argument array by m
        // would be a load from memory, and a wait for it, in every column)
        const int dir = (int)((dir_codes >> (2u * m)) & 3u) - 1;
        const bool prim = m == a.primary;
        // Missing samples take the median's place once it is known: their score is then the +0
        // that a missing sample counts with, and (with a threshold that is not negative) never
        // exceeds, so that the column is scored like any other.  Of a primary metric that
        // falls the zero would be negative; signs leave the fast routes anyway.
        auto missing_stay = [&](float median) {
            return !(a.thr >= 0.0f && a.node_agg == 0 && (!prim || dir >= 0) && median < 3.0e38f);
        };
        // The column's median and MAD go out, and what the score loop needs of them is worked out, by the
        // first wave: done by every wave, the same hundred and thirty instructions kept all four
        // waves of a SIMD busy one after another (2 100 of 41 000 cycles a column at 65 536 ranks).
        auto work_out = [&](float med, float mad, bool special) {
            const ScoreRules rules = sh.rules;
            const float thr = uniform(rules.thr), node_scale = uniform(rules.node_scale), inv_node_scale = rules.inv_node_scale;
            const uint32_t agg = rfl(rules.agg);
            float s = 1.4826f * mad;
            s = fmaxf(s, rules.rel_floor * fabsf(med));
            s = fmaxf(s, rules.abs_floor);

            // The reciprocal route is exact while no intermediate can leave the normal
            // range: all x in [0, 2^59], 2^-34 <= med, 2^-60 <= s <= 2^60 (then every
            // non-zero |x - med| lies in [2^-59, 2^59]).
            const bool exact_recip = !special && umax <= 0x5D000000u && med >= 0x1p-34f && s >= 0x1p-60f &&
                                     s <= 0x1p60f;
            const bool fast = exact_recip && agg == 0;
            // Decision-only route for supporting one-sided metrics: find the exact boundary
            // xstar of "this rank exceeds" by probing 64 consecutive floats around
            // med +- thr*s with the defining operations (IEEE subtract and divide).
            bool decide = fast && !prim && dir != 0 && node_scale > 0.0f;
            float xstar = 0.0f;
            // One vector division serves both: lanes 0..62 probe 63 consecutive floats around
            // med +- thr*s, lane 63 divides 1 by s (the reciprocal every exact route needs).
            const float ss = dir < 0 ? -s : s;
            float rs;
            {
                const float xc = dir > 0 ? med + thr * s : med - thr * s;
                const uint32_t kc = key_of(xc);
                decide = decide && kc >= 64u && kc <= 0xFF800000u - 64u;
                const float xl = float_of_key(kc + (uint32_t)lane - 31u);
                const float num = lane == WAVE - 1 ? 1.0f : (dir > 0 ? xl - med : med - xl);
                const float q = num / s;
                const float r1 = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(q), WAVE - 1));
                rs = dir < 0 ? -r1 : r1;                         // 1/(-s) = -(1/s) exactly
                if (decide) {
                    const uint64_t probes = ~(1ull << (WAVE - 1));
                    const uint64_t mk = gd_ballot(q > thr) & probes;
                    // higher is worse: lanes f..62 true; lower is worse: lanes 0..f-1 true
                    const uint64_t want = dir > 0 ? mk : ~mk & probes;
                    const int f = want ? __builtin_ctzll(want) : 64;
                    decide = f >= 1 && f <= 62 && want == ((~0ull << f) & probes);
                    if (decide) xstar = __uint_as_float((uint32_t)__builtin_amdgcn_readlane(
                                    (int)__float_as_uint(xl), dir > 0 ? f : f - 1));
                    decide = decide && xstar > 0.0f;             // (the bit-pattern comparison needs a positive boundary)
                }
            }
            // decision-only route:
            // |estimate - exact node score| < |cc| * (sum(x) + 8*med) * 2^-20 + |thr| * 2^-23
            // and sum(x) + 8*med <= 16 * max(x):
            const float cc = node_scale * rs;
            const float kk = (8.0f * med) * cc;
            const float margin = __builtin_fmaf(fabsf(cc) * __uint_as_float(umax), 0x1.01p-16f,
                                                fabsf(thr) * 0x1p-22f);
            // The bound on sum(x) beyond which the estimate stays under thr - margin: solved
            // from the estimate's formula (1/cc = ss / node_scale, closely enough) with a little
            // slack and then checked with the formula itself (the estimate rises with the sum when
            // higher is worse, cc > 0, and falls with it otherwise).  Without a bound that passes
            // the check every row is a candidate.
            float sthr = __uint_as_float(opaque_s(dir > 0 ? 0xFF800000u : 0x7F800000u));
            if (decide) {
                const float tl = (thr - margin) - fabsf(thr) * 0x1p-20f;
                const float s0 = (tl + kk) * (ss * inv_node_scale);
                const float slack = fabsf(s0) * 0x1p-18f + 0x1p-100f;
                const float sb = dir > 0 ? s0 - slack : s0 + slack;
                if (__builtin_fmaf(sb, cc, -kk) < tl) sthr = sb;
            }
            const uint32_t shi = sthr >= 0.0f ? __float_as_uint(sthr + 0.0f) : (dir > 0 ? 0u : 0xFFFFFFFFu);
            const uint32_t xcut = dir > 0 ? __float_as_uint(xstar) : ~__float_as_uint(xstar), scut = dir > 0 ? shi : ~shi;
            // 0/1 decision-only (higher / lower is worse), 2/3 exact by reciprocal
            // (one- / two-sided), 4/5 IEEE division (scaled sum / max)
            const uint32_t route = fast ? (decide ? (dir > 0 ? 0u : 1u) : (dir != 0 ? 2u : 3u))
                                        : (agg == 0 ? 4u : 5u);
            if (lane == 0) {
                ScoreParams& p = sh.par;
                p.s = s; p.ss = ss; p.rs = rs; p.cc = cc;
                p.kk = kk; p.margin = margin; p.scut = scut; p.xcut = xcut;
                p.route = route; p.exact_recip = exact_recip ? 1u : 0u;
                p.med = med; p.mad = mad; p.settled = 1;
            }
        };
        // The hinted selection (sign-free column, a predecessor's bracket and MAD): one pass counts, one
        // gathers what may be the median or the MAD, and the first wave alone takes these from the few
        // dozen candidates and works out the column's scoring parameters.  Whatever that does not
        // settle goes through the general route below.
        bool tried_fast = false, settled = false;
        uint32_t located = PLAN_NONE;
        if (hinted && rfl(sh.hfast[m]) != 0 && bracket_counts<LOG_NB>(hint_lo, hint_hi)) {
            tried_fast = true;
            const GatherResult gr = hinted_gather<NT, ROWS, LOG_NB>(
                sh, v, [&](int j) { set_padding(j, tl); }, [&]() { load_ahead(next_col); }, hint_lo, hint_hi, sh.hmad[m], k0_all, k1_all, umax_slot);
            umax = gr.umax;
            located = gr.status;
            if (located != PLAN_NONE) missing = gr.present;
            if (located == PLAN_GATHER) {
                if (w == 0) {
                    float mad = 0.0f;
                    const uint32_t k0 = missing ? (missing - 1) / 2 : k0_all, k1 = missing ? missing / 2 : k1_all;
                    if (finish_gather(sh, lane, k0, k1, &med, &mad)) {
                        if (tid == 0) {             // follow median and MAD step by step
                            sh.hmed[m] = med;
                            sh.hmad[m] = mad;
                            if (boot) { sh.hwl[m] = 1.25f * mad; sh.hwh[m] = 1.25f * mad; }
                        }
                        work_out(med, mad, missing != 0 && missing_stay(med));
                    } else if (lane == 0) {
                        sh.par.settled = 0;
                    }
                }
                __syncthreads();
                settled = rfl(sh.par.settled) != 0;
                med = uniform(sh.par.med);
                special = missing != 0 && missing_stay(med);
            }
        }
        if (__builtin_expect(!settled, 0)) {
        uint32_t s0 = 0, s1 = 0;
        bool have_mad = false;
        int hsel = 0;
        uint32_t listed = 0;                    // distances still to be sorted by the first wave
        if (tried_fast && located == PLAN_NONE) {
            hinted = false;                     // (and this metric goes the general way from now on,
                                                // unless the hint was only a sample's)
            if (tid == 0 && !boot) sh.hfast[m] = 0;
        } else if (tried_fast) {
            const uint32_t k0 = missing ? (missing - 1) / 2 : k0_all, k1 = missing ? missing / 2 : k1_all;
            const HintedResult hr = hinted_rest<NT, ROWS, LOG_NB>(sh, v, sh.hmad[m], k0, k1);
            hsel = hr.found;
            med = 0.5f * (__uint_as_float(hr.m0) + __uint_as_float(hr.m1));
            have_mad = hsel == 2;
            s0 = hr.q0; s1 = hr.q1;
            if (have_mad) listed = hr.listed;
            if (tid == 0) sh.hmed[m] = med;
        }
        // Largest raw bit pattern of the column: >= 0x80000000 iff some value carries
        // a sign bit (negative or -0); otherwise it is the bit pattern of the maximum.
        // With a hint the column is taken to be sign-free like its predecessor and the
        // maximum is found by the median's counting pass itself, which starts on the
        // register rows as they arrive; otherwise it takes a pass of its own.
        const bool fused_umax = FULL && hinted && !tried_fast;
        if (__builtin_expect(!fused_umax && !tried_fast, 0)) {
            uint32_t um = 0;
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
                um = max(um, max(__float_as_uint(v[j][0]), __float_as_uint(v[j][1])));
                um = max(um, max(__float_as_uint(v[j][2]), __float_as_uint(v[j][3])));
                set_padding(j, tl);
            }
            um = wave_max_to_last(um);
            if (lane == WAVE - 1) atomicMax(umax_slot, um);
            __syncthreads();
            umax = rfl(*umax_slot);
        }
        // special: some value carries a sign bit or is a NaN.  The raw bits are then no
        // keys to select by, and a NaN is a missing sample that the ranks must not count.
        special = umax > 0x7F800000u;
        uint32_t k0 = k0_all, k1 = k1_all;

        if (hsel == 0 && !special) {
            uint32_t hlo = 0, hhi = 0;
            int hshift = 0;
            const bool one_round = block_select<NT, ROWS, LOG_NB, true>(
                sh, XKeys<ROWS, true>{v}, __float_as_uint(v[0][0]), true, nsample, k0_all, k1_all, &s0,
                &s1, &hlo, &hhi, &hshift, hinted, hint_lo, hint_hi, fused_umax ? umax_slot : nullptr, &umax);
            special = umax > 0x7F800000u;      // (only the fused pass can find this out here)
        if (!special) {
            med = 0.5f * (__uint_as_float(s0) + __uint_as_float(s1));
            if (one_round)
                have_mad = mad_from_histogram<NT, ROWS, LOG_NB>(sh, v, med, hlo, hhi, hshift, k0_all, k1_all,
                                                                hinted ? sh.hmad[m] : 0.0f, &s0, &s1);
            if (tid == 0) {
                if (have_mad) {                 // keep the reach, follow the median
                    if (!hinted) {
                        // the reach kept for the coming steps: median -+ 1.25 MAD (the edge
                        // pairing looks up to 1.125 MAD away) rather than the sample's wider
                        // bracket -- fewer keys to count, finer buckets, fewer candidates
                        const float madv = 0.5f * (__uint_as_float(s0) + __uint_as_float(s1));
                        sh.hwl[m] = fminf(med - __uint_as_float(hlo), 1.25f * madv);
                        sh.hwh[m] = fminf(__uint_as_float(hhi) - med, 1.25f * madv);
                    }
                    sh.hmed[m] = med;
                    sh.hmad[m] = 0.5f * (__uint_as_float(s0) + __uint_as_float(s1));
                    sh.hok[m] = 1;
                } else {
                    sh.hok[m] = 0;
                }
            }
        }
        }
        uint32_t present = R;
        if (__builtin_expect(missing != 0, 0)) { present = missing; k0 = (present - 1) / 2; k1 = present / 2; }
        if (__builtin_expect(special, 0)) {
            if (tid == 0) sh.hok[m] = 0;
            __syncthreads();    // (a counting pass given up above has just reset its counters)
            // median and MAD are taken over the samples present alone (padding lanes hold NaNs
            // too): the middle one(s) of `present`
            uint32_t top;
            count_present(sh, v, &present, &top);
            __syncthreads();
            if (umax < 0x80000000u) { umax = top; missing = present; }      // (no signs)
            k0 = present ? (present - 1) / 2 : 0u;
            k1 = present / 2;
            if (present) {
                const bool sv = v[0][0] == v[0][0];
                block_select<NT, ROWS, LOG_NB, false>(sh, XKeys<ROWS, false>{v}, key_of(v[0][0] + 0.0f),
                                                      sv, nsample, k0, k1, &s0, &s1);
                // (an odd count has one middle value: no sum that could overflow)
                med = k0 == k1 ? float_of_key(s0) : 0.5f * (float_of_key(s0) + float_of_key(s1));
            }
        }
        if (__builtin_expect(!have_mad && present, 0))
            block_select<NT, ROWS, LOG_NB, false>(sh, DKeys<ROWS>{v, med},
                                                  __float_as_uint(fabsf(v[0][0] - med)),
                                                  v[0][0] == v[0][0], nsample, k0, k1, &s0, &s1);
        if (!present) med = __uint_as_float(opaque_s(0x7FC00000u));  // nothing to take a median of
        if (__builtin_expect(missing != 0, 0)) special = missing_stay(med);
        if (w == 0) {
            if (listed != 0) {
                const uint32_t key = sh.cand[lane];
                const uint32_t sorted = gd_sort64<true>((uint32_t)lane < listed ? key : 0xFFFFFFFFu);
                s0 = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(s0 & (WAVE - 1)));
                s1 = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(s1 & (WAVE - 1)));
            }
            float mad = k0 == k1 ? __uint_as_float(s0) : 0.5f * (__uint_as_float(s0) + __uint_as_float(s1));
            if (!present) mad = __uint_as_float(opaque_s(0x7FC00000u));      // nothing to take a median of
            if (tid == 0) {
                if (hsel) sh.hmad[m] = mad;         // the hinted selection follows median and MAD step by step
                // a column with missing samples, but no signs, leads the next step's selection too
                if (hsel == 0 && missing != 0 && med > 0.0f && mad > 0.0f && med < 3.0e38f && mad < 3.0e38f) {
                    sh.hmed[m] = med; sh.hmad[m] = mad;
                    sh.hwl[m] = 1.25f * mad; sh.hwh[m] = 1.25f * mad;
                    sh.hok[m] = 1;
                }
                // (from here on the reach is the exact MAD's, as after the general route)
                if (boot && hsel == 2) { sh.hwl[m] = 1.25f * mad; sh.hwh[m] = 1.25f * mad; }
            }
            work_out(med, mad, special);
        }
        __syncthreads();
        if (tid == 0) {          // (a zero made here: kept in registers for the whole kernel it ends up spilled)
            const uint32_t zero = opaque_v(0u);
            sh.nkept = zero; sh.nnear = zero;
        }
        for (uint32_t i = opaque_v((uint32_t)tid); i < CAND_REST; i += NT) sh.cand[i] = CAND_NONE;
        load_ahead(next_col);       // (a second time where the hinted selection asked for these rows: they are not kept on this way)
        }
        if (__builtin_expect(missing != 0, 0)) {
          if (!special) {
            const uint32_t absm = opaque_s(0x7FFFFFFFu);
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][i] = (__float_as_uint(v[j][i]) & absm) <= 0x7F800000u ? v[j][i] : med;
                __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
        if (tid == 0) {
            const gd_args_ptr here = args_here();
            here->med[t * M + m] = sh.par.med;
            here->mad[t * M + m] = sh.par.mad;
        }
        // z, exceedance and node scores
        const uint32_t tz = fresh_tid4();
        // (the run-time test that is always true keeps the block a region of its own for the
        // register allocator, as it was when the output pointer decided: without it this
        // instantiation spills)
        if (WANT_Z && opaque_s(1u) != 0u) {   // optional full z output, recomputed so that the loops below stay lean
                     // (it must come first: they refill the registers with the next column)
            float* zcol = args_here()->z + (t * M + m) * (size_t)R;
            // the quotient by the column's reciprocal and two residual corrections where that
            // is exact (see score_row_fast; no sign bits there, so no -0 to read as +0)
            const bool by_recip = opaque_s(sh.par.exact_recip) != 0u;
            // (optimiser-opaque copies of the median and the scale: the differences x - med of
            // this loop must not be kept for the score loop below, 64 registers' worth)
            const float medz = __uint_as_float(opaque_s(__float_as_uint(med)));
            const float sz = __uint_as_float(opaque_s(__float_as_uint(sh.par.s)));
            const float rz = __uint_as_float(opaque_s(__float_as_uint(dir < 0 ? -sh.par.rs : sh.par.rs)));      // 1 / s
            auto quotient = [&](float x) -> float {
                const float d = x - medz;
                const float q0 = d * rz;
                const float e0 = __builtin_fmaf(-q0, sz, d);
                const float q1 = __builtin_fmaf(e0, rz, q0);
                const float e1 = __builtin_fmaf(-q1, sz, d);
                return __builtin_fmaf(e1, rz, q1);
            };
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
                if (holds(j, tz)) {
                    float4 q;
                    if (by_recip) {
                        q.x = quotient(v[j][0]); q.y = quotient(v[j][1]);
                        q.z = quotient(v[j][2]); q.w = quotient(v[j][3]);
                    } else {
                        q.x = ((v[j][0] + 0.0f) - medz) / sz; q.y = ((v[j][1] + 0.0f) - medz) / sz;
                        q.z = ((v[j][2] + 0.0f) - medz) / sz; q.w = ((v[j][3] + 0.0f) - medz) / sz;
                    }
                    if (special) {              // a missing sample (NaN) scores 0
                        const uint32_t absm = opaque_s(0x7FFFFFFFu);
                        q.x = (__float_as_uint(v[j][0]) & absm) <= 0x7F800000u ? q.x : 0.0f;
                        q.y = (__float_as_uint(v[j][1]) & absm) <= 0x7F800000u ? q.y : 0.0f;
                        q.z = (__float_as_uint(v[j][2]) & absm) <= 0x7F800000u ? q.z : 0.0f;
                        q.w = (__float_as_uint(v[j][3]) & absm) <= 0x7F800000u ? q.w : 0.0f;
                    }
                    store_once(zcol + rbase(j, tz), q.x, q.y, q.z, q.w);
                }
                __builtin_amdgcn_sched_barrier(0);      // row by row: nothing of a later row starts early
            }
        }
        const gd_args_ptr here = args_here();
        const float thr = here->thr, node_scale = here->node_scale;
        float* nzrow = here->node_z + t * N;
        const ScoreParams& par = sh.par;
        const float s = uniform(par.s), ss = uniform(par.ss), rs = uniform(par.rs);
        const float cc = uniform(par.cc), kk = uniform(par.kk), margin = uniform(par.margin);
        const uint32_t route = rfl(par.route);
        const uint32_t mask_m = 0x01010101u << m;
        __builtin_amdgcn_s_setprio(0);
        uint32_t* const emask_lane = emask + opaque_v((uint32_t)tid);      // (row j: a constant offset from here)
        auto done_with = [&](int j, uint32_t eplaced) {
            __hip_atomic_fetch_or(&emask_lane[j * NT], eplaced, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            // the row is done: refill it with the next column
            if (j < AHEAD) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[j][i] = ahead[j < AHEAD ? j : 0][i];
            } else if (!SPLIT && j < EARLY) load_row(j, next_col, tz);
            // pin the row's results here, or its scores stay live until the loop ends
            asm volatile("" : "+v"(NE[j / 4]));
            __builtin_amdgcn_sched_barrier(0);
        };
        const uint32_t flip = route == 0u ? 0xFFFFFFFFu : 0u;
        const uint32_t xcut = opaque_v(par.xcut), scut = opaque_v(par.scut);      // (vector registers: an instruction takes one scalar)
        const uint32_t absmask = dir == 0 ? 0x7FFFFFFFu : 0xFFFFFFFFu;
        const uint32_t sgnmask = dir < 0 ? 0x80000000u : 0u;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const uint32_t rt = opaque_s(route);
            uint32_t eplaced;
            if (rt <= 1u) {
                const float half = (v[j][0] + v[j][1]) + (v[j][2] + v[j][3]);
                const float sum = half + lane_xor1(half);
                if (__builtin_expect(gd_ballot((int32_t)decided(sum, flip, scut) < 0) != 0, 0)) {
                    // some node may exceed: the estimate decides, or, too close, the exact chain (padding, NaNs, comes
                    // here where higher is worse: the NaN exceeds nothing)
                    float nz = __builtin_fmaf(sum, cc, -kk);
                    if (__builtin_expect(gd_ballot(fabsf(nz - thr) <= margin) != 0, 0)) {
                        uint32_t e2;
                        score_row_fast<false>(v[j], med, ss, rs, thr, node_scale, mask_m, &e2, &nz);
                    }
                    NE[j / 4] |= (nz > thr ? 1u : 0u) << (8 * (j & 3) + m);
                }
                eplaced = sign_bytes(decided(v[j][0], flip, xcut), decided(v[j][1], flip, xcut),
                                     decided(v[j][2], flip, xcut), decided(v[j][3], flip, xcut), mask_m);
            } else {
                float nz;
                if (rt == 2u) {
                    score_row_fast<false>(v[j], med, ss, rs, thr, node_scale, mask_m, &eplaced, &nz);
                } else if (rt == 3u) {
                    score_row_fast<true>(v[j], med, ss, rs, thr, node_scale, mask_m, &eplaced, &nz);
                } else {
                    uint32_t e;
                    score_row(rt - 4u, v[j], med, s, absmask, sgnmask, thr, node_scale, &e, &nz);
                    eplaced = e << m;
                }
                NE[j / 4] |= (nz > thr ? 1u : 0u) << (8 * (j & 3) + m);
                if (prim && holds(j, tz) && !(tz & 4)) nzrow[rbase(j, tz) / 8] = nz;
            }
            done_with(j, eplaced);
        }
#pragma unroll
        for (int j = EARLY; j < ROWS; ++j) load_row(j, next_col, tz);
    }

    const uint32_t to = fresh_tid4();
    const gd_args_ptr out = args_here();
    const uint32_t primary = out->primary;
    uint8_t* erow = out->exceed_mask + t * R;
    if (SPLIT) {
        // This column's exceed bits go out as bit planes, for combine_kernel to put together:
        // those of PLANE_RANKS ranks as M planes in the mask bytes of these ranks, those of
        // their nodes in their anomaly words (eight planes fit either).
        // Rows in pairs and fours, so that every lane stores a byte: written row by row, by half of
        // the lanes and by one in sixteen, one step of 65 536 ranks x 8 took 29.3 us (now 27.3; 26.1
        // with the atomics that needed the masks cleared first), of 16 384 x 8 16.1 (15.6).
        static_assert(!SPLIT || ROWS % 2 == 0, "rows in pairs");
        uint8_t* const wrow8 = reinterpret_cast<uint8_t*>(out->rank_anom + t * RW);
        const bool odd = (to & 4u) != 0;                 // (lanes 2p and 2p + 1: one node's ranks)
        auto nibble_bits = [&](int j) {                  // bit 0 of each byte: the rank exceeds
            return holds(j, to) ? (emask[j * NT + to / 4] >> m_begin) & 0x01010101u : 0u;
        };
#pragma unroll
        for (int j = 0; j < ROWS; j += 2) {
            // this lane's ranks of both rows, four bits each; even lanes store row j, odd ones row j + 1
            const uint32_t own = __builtin_amdgcn_udot4(nibble_bits(j), 0x08040201u,
                                                        __builtin_amdgcn_udot4(nibble_bits(j + 1), 0x80402010u, 0u, false),
                                                        false);
            const uint32_t other = lane_xor<1>(own);
            const uint32_t byte = odd ? (other >> 4) | (own & 0xF0u) : (own & 0xFu) | (other << 4);
            const uint32_t r = (odd ? block_of(j + 1) : block_of(j)) * BLK + (to & ~4u);
            const uint32_t r0 = r & ~(PLANE_RANKS - 1u), here = min(PLANE_RANKS, R - r0);
            if (j + 1 < TAIL || r < R) erow[r0 + (m_begin * here + (r - r0)) / 8] = (uint8_t)byte;
        }
#pragma unroll
        for (int q = 0; q < (ROWS + 3) / 4; ++q) {
            // eight nodes, the even ones of sixteen lanes, make a byte; four rows' bytes at once
            uint32_t nb = (NE[q] >> m_begin) & 0x01010101u;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * q + i < ROWS && !holds(4 * q + i, to)) nb &= ~(0xFFu << (8 * i));
            const uint32_t place = (to >> 3) & 7u;
            nb = odd ? 0u : nb << place;
            nb |= lane_xor<2>(nb);
            nb |= lane_xor<4>(nb);
            nb |= lane_xor<8>(nb);
            const uint32_t row = 4 * q + place;          // (the byte that this lane stores)
            if (!odd && place < 4u && row < (uint32_t)ROWS) {
                const uint32_t r = block_of((int)row) * BLK + (to & ~63u);
                const uint32_t r0 = r & ~(PLANE_RANKS - 1u), here = min(PLANE_RANKS, R - r0);
                if (r < R)
                    wrow8[r0 / 8 + m_begin * ((here + 63) / 64) + (r - r0) / 64] = (uint8_t)(nb >> (8 * place));
            }
        }
        return;
    }
    // per-rank mask bytes and anomaly bits.  Anomalous ranks are rare: their bits are OR-ed
    // into the step's bit words in LDS (all zero between steps) only by the waves that
    // hold one, and the finished words are copied out below.
    const uint32_t min_signals = rfl(out->min_signals), others_mask = ~(0x01010101u << primary);
    // multi-signal rule on four mask bytes at once: primary bit set and at least min_signals
    // bits in the byte; the answer is bit 0 of each byte
    auto rule4 = [&](uint32_t E) -> uint32_t {
        const uint32_t prim_set = (E >> primary) & 0x01010101u;
        if (min_signals <= 2u) {
            // (two signals: the primary's and any other -- bit 7 of "low seven bits + 0x7F",
            // or bit 7 itself, says that a byte is not zero)
            const uint32_t others = E & others_mask;
            const uint32_t some = (((others & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | others) >> 7;
            return min_signals <= 1u ? prim_set : (prim_set & some);
        }
        // per-byte popcount >= min_signals (adding 0x80 - min_signals carries into bit 7)
        uint32_t pc = E - ((E >> 1) & 0x55555555u);
        pc = (pc & 0x33333333u) + ((pc >> 2) & 0x33333333u);
        pc = (pc + (pc >> 4)) & 0x0F0F0F0Fu;
        return prim_set & ((pc + (0x80u - min_signals) * 0x01010101u) >> 7);
    };
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const bool valid = holds(j, to);
        const uint32_t Ej = emask[j * NT + to / 4];
        if (valid) store_once(reinterpret_cast<uint32_t*>(erow + rbase(j, to)), Ej);
        uint32_t an = rule4(Ej);
        if (!valid) an = 0u;
        if (__builtin_expect(gd_ballot(an != 0u) != 0ull, 0)) {
            // the lane's four ranks are bits rbase % 32 .. + 3 of 32-bit word rbase / 32
            const uint32_t nib = (an | (an >> 7) | (an >> 14) | (an >> 21)) & 0xFu;
            const uint32_t r0 = rbase(j, to);
            if (nib) atomicOr(&reinterpret_cast<uint32_t*>(sh.ranka)[r0 >> 5], nib << (r0 & 31u));
        }
        if (valid && !(to & 4)) sh.nodeb[rbase(j, to) / 8] = (uint8_t)((NE[j / 4] >> (8 * (j & 3))) & 0xFFu);
    }
    __syncthreads();
    for (uint32_t q = tid; q < RW; q += NT) {       // (one round at most in the exact-fit tilings)
        out->rank_anom[t * RW + q] = sh.ranka[q];
        sh.ranka[q] = 0;
    }
    if (ROWS >= 10) {
        // Eight nodes per thread (N <= 8 * NT): one 8-byte read of the staged bytes and, where
        // the step's bytes begin at a multiple of eight, one 8-byte store; the rule
        // byte-parallel as for the ranks; eight consecutive lanes make one 64-bit anomaly word
        const uint32_t tq = opaque_v((uint32_t)tid), sl = tq & 7u;
        uint2 nb = *reinterpret_cast<const uint2*>(&sh.nodeb[min(8 * tq, (uint32_t)MAX_NODES - 8)]);
        uint8_t* nm = out->node_mask + t * N + 8 * tq;
        const uint32_t here = FULL ? 8u : (8 * tq < N ? min(N - 8 * tq, 8u) : 0u);      // (nodes of this thread)
        if (!FULL && here < 8) {                // (bytes beyond the last node were never written)
            nb.x &= here >= 4 ? 0xFFFFFFFFu : (1u << (8 * here)) - 1u;
            nb.y &= here <= 4 ? 0u : (1u << (8 * (here - 4))) - 1u;
        }
        if (here == 8 && ((uintptr_t)(out->node_mask + t * N) & 7u) == 0) {
            *reinterpret_cast<uint2*>(nm) = nb;
        } else {
#pragma unroll
            for (uint32_t i = 0; i < 8; ++i)
                if (FULL || i < here) nm[i] = (uint8_t)((i < 4 ? nb.x : nb.y) >> (8 * (i & 3)));
        }
        const uint32_t a0 = rule4(nb.x), a1 = rule4(nb.y);
        const uint32_t ab = ((a0 | (a0 >> 7) | (a0 >> 14) | (a0 >> 21)) & 0xFu) |
                            (((a1 | (a1 >> 7) | (a1 >> 14) | (a1 >> 21)) & 0xFu) << 4);
        uint32_t wlo = sl < 4u ? ab << (8u * sl) : 0u;
        uint32_t whi = sl >= 4u ? ab << (8u * (sl - 4u)) : 0u;
        wlo |= lane_xor<1>(wlo); whi |= lane_xor<1>(whi);
        wlo |= lane_xor<2>(wlo); whi |= lane_xor<2>(whi);
        wlo |= lane_xor<4>(wlo); whi |= lane_xor<4>(whi);
        if (sl == 0u && (FULL || 8 * tq < N)) out->node_anom[t * NWD + tq / 8u] = ((uint64_t)whi << 32) | wlo;
    } else {
        if (FULL) {                             // N == NT * ROWS / 2: a fixed number of rounds
#pragma unroll
            for (int q = 0; q < (ROWS + 1) / 2; ++q) {
                const uint32_t n = opaque_v((uint32_t)tid) + (uint32_t)q * NT;
                if (ROWS % 2 == 0 || n < N) out->node_mask[t * N + n] = sh.nodeb[n];
            }
        } else {
            for (uint32_t n = tid; n < N; n += NT) out->node_mask[t * N + n] = sh.nodeb[n];
        }
        for (uint32_t wd = w; wd < NWD; wd += NWAVES) {
            const uint32_t n = wd * 64 + lane;
            bool an = false;
            if (n < N) {
                const uint32_t b = sh.nodeb[n];
                an = ((b >> primary) & 1u) && (uint32_t)__popc(b) >= out->min_signals;
            }
            const uint64_t word = gd_ballot(an);
            if (lane == 0) out->node_anom[t * NWD + wd] = word;
        }
    }
    }   // steps of this workgroup
}

#include "score_small.h"

// NT threads per column (64: one wave per column, M of them per workgroup; LOG_NB has no
// meaning there).  <= 128 VGPRs: 16 waves per CU.
constexpr int block_threads(int NT) { return NT == WAVE ? 8 * WAVE : NT; }
// Waves per SIMD.  Up to eight rows of 256 threads are kept to 96 VGPRs, and five such workgroups fit
// a CU's LDS: their time is mostly that of the short phases, which overlap (four / five: 10 000
// steps, 4 096 ranks x 1 141 / 127 us, 5 000 x 8 784 / 677, 6 000 x 4 456 / 399, 8 000 x 4 491 / 440;
// 1 200 steps, which four to a CU take in two rounds, 8 000 x 4 94 / 68).  The ragged tiling of eight
// rows has two registers too many for that and keeps them in scratch memory, 12 bytes a lane: up to
// 1 024 steps, where there is no fifth to run, 8 000 ranks take 1 % longer so (x 8 102.5 / 103.8).
constexpr int waves_of(int nt, int rows, bool want_z) { return nt == 256 && rows <= 8 && !want_z ? 5 : 4; }
template <int NT, int ROWS, int LOG_NB, bool FULL, bool SPLIT, bool WANT_Z>
__global__ __launch_bounds__(block_threads(NT), waves_of(NT, ROWS, WANT_Z)) void score_kernel(const gd_score_args a) {
    if constexpr (NT == WAVE) score_small<ROWS, FULL, WANT_Z>(a);
    else score_columns<NT, ROWS, LOG_NB, FULL, SPLIT, WANT_Z>(a);
}
template <int NT, int ROWS, int LOG_NB, bool SPLIT, bool WANT_Z>
__global__ __launch_bounds__(block_threads(NT), waves_of(NT, ROWS, WANT_Z)) void score_ragged_kernel(const gd_score_args a) {
    if constexpr (NT == WAVE) score_small<ROWS, false, WANT_Z>(a);
    else score_columns<NT, ROWS, LOG_NB, false, SPLIT, WANT_Z>(a);
}
template <int NT, int ROWS, int LOG_NB, bool FULL, bool SPLIT>
constexpr auto kernel_of() {
    if constexpr (FULL) return &score_kernel<NT, ROWS, LOG_NB, true, SPLIT, WANT_Z_HERE>;
    else return &score_ragged_kernel<NT, ROWS, LOG_NB, SPLIT, WANT_Z_HERE>;
}

// Eight bytes of eight bits: bit j of byte i becomes bit i of byte j.
__device__ __forceinline__ uint64_t transpose8x8(uint64_t x) {
    uint64_t t = (x ^ (x >> 7)) & 0x00AA00AA00AA00AAull;
    x ^= t ^ (t << 7);
    t = (x ^ (x >> 14)) & 0x0000CCCC0000CCCCull;
    x ^= t ^ (t << 14);
    t = (x ^ (x >> 28)) & 0x00000000F0F0F0F0ull;
    return x ^ t ^ (t << 28);
}

// Split route, after the columns: mask bytes and anomaly words from the columns' bit planes,
// which lie where they go (see score_columns): a workgroup has read all the planes of its
// PLANE_RANKS ranks, a thread those of eight, when it writes the first byte.  Latency-bound
// (one round of loads, one of stores).  The planes spare the zeroing launch and the atomics
// that merged the columns' bits before (one step of 32 768 ranks x 8: 2.0 + 14.4 + 4.0 us in
// three launches, now 15.8 + 4.0 in two), and whole words per step, without which a call took the
// route of long batches (14 072 x 8: 118 -> 26 us a call).  One workgroup per step, which
// needs no order of the planes, took 12 us for this.
__global__ __launch_bounds__(PLANE_RANKS / 8) void combine_kernel(const gd_score_args a) {
    const uint32_t tid = threadIdx.x, sl = tid & 7u, R = a.R, N = a.N, M = a.M;
    const uint32_t RW = (R + 63) / 64, NWD = (N + 63) / 64;
    const uint32_t r0 = blockIdx.x * PLANE_RANKS, here = min(PLANE_RANKS, R - r0);
    const uint32_t groups = here / 8, nbytes = (here + 63) / 64;      // (eight ranks, one node each; bytes of a node plane)
    const size_t t = blockIdx.y;
    uint8_t* const mask = a.exceed_mask + t * R + r0;
    uint64_t* const words = a.rank_anom + t * RW + r0 / 64;
    uint64_t ranks = 0, nodes = 0;                              // byte m: plane m
#pragma unroll
    for (uint32_t m = 0; m < 8; ++m) {
        if (m < M && tid < groups) ranks |= (uint64_t)mask[m * groups + tid] << (8 * m);
        if (m < M && tid < nbytes) nodes |= (uint64_t)reinterpret_cast<const uint8_t*>(words)[m * nbytes + tid] << (8 * m);
    }
    // (every load has arrived before the first store of any wave)
    asm volatile("" : "+v"(ranks), "+v"(nodes));
    __syncthreads();
    const uint32_t min_signals = a.min_signals, primary = a.primary;
    // the rule on eight bytes: bit j of the answer for byte j
    auto rule8 = [&](uint64_t E) -> uint32_t {
        const uint32_t lo = small_rule4((uint32_t)E, primary, min_signals);
        const uint32_t hi = small_rule4((uint32_t)(E >> 32), primary, min_signals);
        return ((lo | (lo >> 7) | (lo >> 14) | (lo >> 21)) & 0xFu) |
               (((hi | (hi >> 7) | (hi >> 14) | (hi >> 21)) & 0xFu) << 4);
    };
    // eight lanes' bytes make a word
    auto word_of = [&](uint32_t byte) -> uint64_t {
        uint32_t wlo = sl < 4u ? byte << (8u * sl) : 0u, whi = sl >= 4u ? byte << (8u * (sl - 4u)) : 0u;
        wlo |= lane_xor<1>(wlo); whi |= lane_xor<1>(whi);
        wlo |= lane_xor<2>(wlo); whi |= lane_xor<2>(whi);
        wlo |= lane_xor<4>(wlo); whi |= lane_xor<4>(whi);
        return ((uint64_t)whi << 32) | wlo;
    };
    const uint64_t E = transpose8x8(ranks);                     // (0 beyond the last rank)
    const uint64_t w = word_of(rule8(E));
    if (tid < groups) {
        reinterpret_cast<uint32_t*>(mask + 8 * tid)[0] = (uint32_t)E;
        reinterpret_cast<uint32_t*>(mask + 8 * tid)[1] = (uint32_t)(E >> 32);
        if (sl == 0) words[tid / 8] = w;
    }
    const uint64_t F = transpose8x8(nodes);
    const uint64_t v = word_of(rule8(F));
    if (tid < nbytes) {
        uint8_t* const nm = a.node_mask + t * N + r0 / 8 + 8 * tid;      // (at any address)
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
            if (8 * tid + i < groups) nm[i] = (uint8_t)(F >> (8 * i));
        if (sl == 0) a.node_anom[t * NWD + r0 / 512 + tid / 8] = v;
    }
}

// Diagnostic: the scoring kernel's loads and nothing else -- persistent 1024-thread
// workgroups, each reading a contiguous run of 256 KB blocks, sixteen float4 loads
// per thread and block -- as the ceiling that a single pass over the data has.
__global__ __launch_bounds__(1024) void read_probe_kernel(const float* x, uint64_t n_blocks,
                                                          uint32_t* sink) {
    constexpr uint32_t BLOCK_FLOATS = 1024 * 4 * 16;
    const uint64_t per = (n_blocks + gridDim.x - 1) / gridDim.x;
    const uint64_t b0 = blockIdx.x * per, b1 = b0 + per < n_blocks ? b0 + per : n_blocks;
    uint32_t acc = 0;
    for (uint64_t b = b0; b < b1; ++b) {
        const float* p = x + b * BLOCK_FLOATS + threadIdx.x * 4;
        float4 q[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) q[j] = *reinterpret_cast<const float4*>(p + j * 4096);
#pragma unroll
        for (int j = 0; j < 16; ++j)
            acc = max(acc, max(max(__float_as_uint(q[j].x), __float_as_uint(q[j].y)),
                               max(__float_as_uint(q[j].z), __float_as_uint(q[j].w))));
    }
    if (acc == 0xFFFFFFFFu) *sink = acc;      // (keeps the loads alive; NaN patterns aside, never true)
}

int compute_units(hipError_t* err) {
    static std::atomic<int> known{0};        // (several threads may ask at once)
    *err = hipSuccess;
    int n_cu = known.load(std::memory_order_relaxed);
    if (n_cu == 0) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) { *err = e; return 0; }
        if (n_cu <= 0) n_cu = 256;
        known.store(n_cu, std::memory_order_relaxed);
    }
    return n_cu;
}

// One workgroup per column pays off while the columns fit the chip side by side.
bool use_split(const gd_score_args& a, int n_cu) {
    return a.split_steps > 0 && a.T <= a.split_steps && (uint64_t)a.T * a.M <= (uint64_t)n_cu;
}

// Up to 4 096 ranks: one wave per column scores the M columns of a step side by side, 256 threads
// one after another but each column faster.  Measured (us by 256 threads / by waves):
//   1 025 to 2 048 ranks, one metric: 256 steps 18 / 21 (missing samples 16 / 22, both signs 16 / 28,
//     whole degrees 17..165 / 25..52), 1 500 steps 37 / 25; two metrics: 256 steps 31 / 20
//   2 049 to 3 072 ranks, two metrics: 256 steps 29 / 33 (missing 26 / 35, signs 26 / 41, equal values
//     50 / 15, values over decades 170 / 50), 1 500 steps 60 / 43; three: 256 steps 42 / 34
//   3 073 to 4 096 ranks, two metrics: 500 steps 36 / 43 (missing 35 / 43, signs 32 / 62, few distinct
//     values 68 / 15, decades 180 / 55), 3 000 steps 91 / 82; four: 256 steps 50 / 39, 3 000 155 / 124;
//     one: 2 000 steps 42 / 56 (the lines cross at about 8 000 steps)
// Two metrics and more go to the waves, whose time the contents change least, and one metric up to
// 2 048 ranks.  Of a five- or six-wave workgroup only two fit a CU above 3 072 ranks, where four of
// four waves do: long batches are the 256 threads' there (five metrics, 1 500 steps 135 / 126,
// 3 000 187 / 229; six, 1 500 160 / 132).
bool one_wave_per_column(const gd_score_args& a) {
    if (a.R <= 2048) return true;
    if (a.R > 4096) return false;
    if (a.R > 3072 && (a.M == 5 || a.M == 6)) return a.T <= 1536;
    return a.M > 1;
}

template <int NT, int ROWS, int LOG_NB>
constexpr size_t lds_bytes() {
    using SH = Shared<NT, LOG_NB, NT * 4 * ROWS / 8>;
    return ((sizeof(SH) + 15) & ~(size_t)15) + (size_t)ROWS * NT * 4;
}

// Few ranks: a workgroup per step, a wave per column, in short batches and long ones
// (launched in pieces, because a grid's threads have to fit 32 bits).
template <int ROWS, bool FULL, bool SPLIT>
hipError_t launch_small(gd_score_args a, hipStream_t s) {
    constexpr uint32_t MOST = 1u << 22;
    static_assert(SmallLds<ROWS>::bytes(8) <= 64 * 1024, "LDS that a launch may ask for without more ado");
    for (;;) {
        const uint32_t n = a.T < MOST ? a.T : MOST;
        hipLaunchKernelGGL((kernel_of<WAVE, ROWS, 10, FULL, SPLIT>()), dim3(n), dim3(WAVE * a.M),
                           SmallLds<ROWS>::bytes(a.M), s, a);
        const hipError_t e = hipGetLastError();
        a.T -= n;
        if (e != hipSuccess || a.T == 0) return e;
        const size_t columns = (size_t)n * a.M;
        a.x += columns * a.R; a.med += columns; a.mad += columns;
        if (a.z) a.z += columns * a.R;
        a.exceed_mask += (size_t)n * a.R; a.rank_anom += (size_t)n * ((a.R + 63) / 64);
        a.node_z += (size_t)n * a.N; a.node_mask += (size_t)n * a.N; a.node_anom += (size_t)n * ((a.N + 63) / 64);
    }
}

// A whole batch: enough workgroups to fill every CU once (as many as fit by LDS and
// wave slots); each takes a contiguous run of ceil(T / grid) steps.
template <int NT, int ROWS, int LOG_NB, bool FULL>
hipError_t launch_runs(const gd_score_args& a, int n_cu, hipStream_t s) {
    if constexpr (NT == WAVE) return launch_small<ROWS, FULL, false>(a, s);
    else {
    if (a.R < (uint32_t)NT * 4) return hipErrorInvalidValue;      // (row 0 holds ranks throughout)
    constexpr size_t lds = lds_bytes<NT, ROWS, LOG_NB>();
    static_assert(lds <= 160 * 1024, "LDS budget of one CU");
    auto kern = kernel_of<NT, ROWS, LOG_NB, FULL, false>();
    static std::atomic<uint64_t> granted{0};
    const hipError_t e = gd_grant_lds(granted, reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    const size_t by_lds = (size_t)160 * 1024 / lds, by_waves = (size_t)(4 * waves_of(NT, ROWS, WANT_Z_HERE)) / (NT / WAVE);
    const size_t per_cu = by_lds < by_waves ? (by_lds ? by_lds : 1) : by_waves;
    const size_t cap = (size_t)n_cu * per_cu;
    const uint32_t grid = (uint32_t)(a.T < cap ? a.T : cap);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT), lds, s, a);
    return hipGetLastError();
    }
}

// A short batch: one workgroup per column, then the combining kernel.
template <int NT, int ROWS, int LOG_NB, bool FULL>
hipError_t launch_columns(const gd_score_args& a, hipStream_t s) {
    if constexpr (NT == WAVE) return launch_small<ROWS, FULL, true>(a, s);
    else {
    if (a.R < (uint32_t)NT * 4) return hipErrorInvalidValue;      // (row 0 holds ranks throughout)
    constexpr size_t lds = lds_bytes<NT, ROWS, LOG_NB>();
    static_assert(lds <= 160 * 1024, "LDS budget of one CU");
    auto kern = kernel_of<NT, ROWS, LOG_NB, FULL, true>();
    static std::atomic<uint64_t> granted{0};
    const hipError_t e = gd_grant_lds(granted, reinterpret_cast<const void*>(kern), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.T * a.M), dim3(NT), lds, s, a);
    hipLaunchKernelGGL(combine_kernel, dim3((a.R + PLANE_RANKS - 1) / PLANE_RANKS, a.T), dim3(PLANE_RANKS / 8), 0, s, a);
    return hipGetLastError();
    }
}

#if GD_SCORE_RAGGED == 0

// Exact fit.  NT x ROWS: the tiling of a batch; CNT x CROWS: that of the per-column route,
// where a column has the CU to itself and is spread over more threads (fewer rows per lane:
// shorter passes between the barriers).
template <int NT, int ROWS, int LOG_NB, int CNT = NT, int CROWS = ROWS, int CLOG_NB = LOG_NB>
hipError_t launch(const gd_score_args& a, int n_cu, hipStream_t s) {
    static_assert(NT * ROWS == CNT * CROWS, "both tilings hold the same number of ranks");
    return use_split(a, n_cu) ? launch_columns<CNT, CROWS, CLOG_NB, true>(a, s)
                              : launch_runs<NT, ROWS, LOG_NB, true>(a, n_cu, s);
}

// Pick the register tiling for R: NT threads x ROWS float4 rows hold NT*4*ROWS ranks.
hipError_t pick_tiling(const gd_score_args& a, hipStream_t s) {
    hipError_t e;
    const int n_cu = compute_units(&e);
    if (e != hipSuccess) return e;
    // (the 256-thread tilings take 2048 buckets: four workgroups then share a CU's LDS, and
    // their barrier-bound phases overlap)
    static_assert(4 * lds_bytes<256, 16, 11>() <= 160 * 1024, "four workgroups of the 16 384-rank tiling share a CU's LDS");
    static_assert(5 * lds_bytes<256, 8, 11>() <= 160 * 1024, "five of those of up to 8 192 ranks");
    switch (a.R) {
        case 256: return launch<64, 1, 10>(a, n_cu, s);
        case 1024: return launch<64, 4, 10>(a, n_cu, s);
        case 4096:
            if (one_wave_per_column(a) && !use_split(a, n_cu)) break;
            return launch<256, 4, 11>(a, n_cu, s);
        case 16384: return launch<256, 16, 11, 1024, 4, 12>(a, n_cu, s);
        case 32768: return launch<512, 16, 12, 1024, 8, 12>(a, n_cu, s);
        case 65536: return launch<1024, 16, 12>(a, n_cu, s);
    }
    if (a.R > 65536) return hipErrorInvalidValue;
    constexpr bool z = WANT_Z_HERE;
    // (up to 2 048 ranks a column is one wave's on either route)
    if (a.R > 2048 && use_split(a, n_cu)) return z ? gd_launch_ragged_columns_z(a, s) : gd_launch_ragged_columns(a, s);
    if (a.R <= 8192) return z ? gd_launch_ragged_few_z(a, n_cu, s) : gd_launch_ragged_few(a, n_cu, s);
    return z ? gd_launch_ragged_many_z(a, n_cu, s) : gd_launch_ragged_many(a, n_cu, s);
}

#endif

}  // namespace

#if GD_SCORE_RAGGED == 1 || GD_SCORE_RAGGED == 2 || GD_SCORE_RAGGED == 3
#if GD_SCORE_WANT_Z
#define GD_RAGGED(name) name##_z
#else
#define GD_RAGGED(name) name
#endif
#endif

// Ragged rank counts: the smallest tiling in steps of two rows, so that no more than the
// last two rows hold padding (one wave per column checks every row).
#if GD_SCORE_RAGGED == 1

hipError_t GD_RAGGED(gd_launch_ragged_few)(const gd_score_args& a, int n_cu, hipStream_t s) {
    const uint32_t R = a.R;
    if (R <= 256) return launch_runs<64, 1, 10, false>(a, n_cu, s);
    if (R <= 512) return launch_runs<64, 2, 10, false>(a, n_cu, s);
    if (R <= 1024) return launch_runs<64, 4, 10, false>(a, n_cu, s);
    if (one_wave_per_column(a)) {
        if (R <= 2048) return launch_runs<64, 8, 10, false>(a, n_cu, s);
        if (R <= 3072) return launch_runs<64, 12, 10, false>(a, n_cu, s);
        return launch_runs<64, 16, 10, false>(a, n_cu, s);
    }
    if (R <= 4096) return launch_runs<256, 4, 11, false>(a, n_cu, s);
    if (R <= 6144) return launch_runs<256, 6, 11, false>(a, n_cu, s);
    return launch_runs<256, 8, 11, false>(a, n_cu, s);
}

#elif GD_SCORE_RAGGED == 2

hipError_t GD_RAGGED(gd_launch_ragged_many)(const gd_score_args& a, int n_cu, hipStream_t s) {
    const uint32_t R = a.R;
    if (R <= 10240) return launch_runs<256, 10, 11, false>(a, n_cu, s);
    if (R <= 12288) return launch_runs<256, 12, 11, false>(a, n_cu, s);
    if (R <= 14336) return launch_runs<256, 14, 11, false>(a, n_cu, s);
    if (R <= 16384) return launch_runs<256, 16, 11, false>(a, n_cu, s);
    if (R <= 20480) return launch_runs<512, 10, 12, false>(a, n_cu, s);
    if (R <= 24576) return launch_runs<512, 12, 12, false>(a, n_cu, s);
    if (R <= 28672) return launch_runs<512, 14, 12, false>(a, n_cu, s);
    if (R <= 32768) return launch_runs<512, 16, 12, false>(a, n_cu, s);
    if (R <= 40960) return launch_runs<1024, 10, 12, false>(a, n_cu, s);
    if (R <= 49152) return launch_runs<1024, 12, 12, false>(a, n_cu, s);
    if (R <= 57344) return launch_runs<1024, 14, 12, false>(a, n_cu, s);
    return launch_runs<1024, 16, 12, false>(a, n_cu, s);
}

#elif GD_SCORE_RAGGED == 3

hipError_t GD_RAGGED(gd_launch_ragged_columns)(const gd_score_args& a, hipStream_t s) {
    const uint32_t R = a.R;
    if (R <= 4096) return launch_columns<256, 4, 11, false>(a, s);
    if (R <= 8192) return launch_columns<1024, 2, 12, false>(a, s);
    if (R <= 16384) return launch_columns<1024, 4, 12, false>(a, s);
    if (R <= 24576) return launch_columns<1024, 6, 12, false>(a, s);
    if (R <= 32768) return launch_columns<1024, 8, 12, false>(a, s);
    if (R <= 40960) return launch_columns<1024, 10, 12, false>(a, s);
    if (R <= 49152) return launch_columns<1024, 12, 12, false>(a, s);
    if (R <= 57344) return launch_columns<1024, 14, 12, false>(a, s);
    return launch_columns<1024, 16, 12, false>(a, s);
}

#elif GD_SCORE_WANT_Z

hipError_t gd_launch_score_with_z(const gd_score_args& a, hipStream_t s) { return pick_tiling(a, s); }

#else

hipError_t gd_launch_read_probe(const float* d_x, uint64_t n_bytes, uint32_t* d_sink, hipStream_t s) {
    const uint64_t n_blocks = n_bytes / (256 * 1024);
    if (n_blocks == 0) return hipSuccess;
    hipError_t e;
    const int n_cu = compute_units(&e);
    if (e != hipSuccess) return e;
    const uint32_t grid = (uint32_t)(n_blocks < (uint64_t)n_cu ? n_blocks : (uint64_t)n_cu);
    hipLaunchKernelGGL(read_probe_kernel, dim3(grid), dim3(1024), 0, s, d_x, n_blocks, d_sink);
    return hipGetLastError();
}

hipError_t gd_launch_score(const gd_score_args& a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    return a.z ? gd_launch_score_with_z(a, s) : pick_tiling(a, s);
}

#endif
