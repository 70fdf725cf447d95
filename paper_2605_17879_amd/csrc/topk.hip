// Ranking of the slowest nodes for the operator: nodes ordered by (window
// count, latest primary node score, node index) -- the nodes Section 4.2 would
// remove from the healthy pool first.
//
// The middle field of the key is the latest primary node score or, for the
// ranking by the score averaged over the window, the window's sum of quantised
// scores.
//
// One workgroup builds a unique 64-bit key per node (N <= 8192) and writes the k
// largest in descending order.  The launch is one chain of dependent steps over 48 KB
// of input, so the length of the chain is what counts.
//
// k <= 64 (the usual request): nothing is sorted.
//   1. A thread loads 1, 2, 4 or 8 neighbouring nodes (three vector loads at the most)
//      and keeps their keys in registers.
//   2. The largest digest (see below: the count and the leading bits of the score) of every
//      group of up to 8 neighbouring threads goes into LDS: 128 to 255 values.  Each wave ranks
//      a few of them against all (one value per lane, a compare and a count of the
//      lanes per 64).  The k-th largest is a threshold that at least k keys reach --
//      it is the k-th largest of a subset -- and, a group's best being the likeliest of
//      its members, few more do (about 90 of 8 192 keys in random order for k = 64).
//   3. The keys that reach it are compacted into LDS and ranked in the same way; a
//      key's rank is its place in the output.  Where very many reach it (equal scores
//      throughout), the k-th largest of the threads' best whole keys is the threshold instead,
//      which at most 8 k keys reach: 8 192 equal scores take 11 us, 70 where they were sorted.
// Measured (launch time, k = 64): 8 192 nodes 12.5 -> 6.1 us, 8 nodes 7.5 -> 2.0 us.
// Before, the waves sorted their threads' largest keys and one wave folded the sixteen
// sorted lists one after another; with that fold replaced by a sort of the waves' best
// eight it was 10.5 us, a sixth of it waiting for sixteen 2- and 4-byte loads per thread.
//
// At most 64 nodes: one wave, one sort by lane exchanges.
// Larger k: all keys are sorted in LDS with a bitonic network.
#include "gd_internal.h"
#include "gd_lanes.h"

namespace {

constexpr int WAVE = 64;
constexpr int TOPK_NT = 1024;
constexpr int TOPK_MAX = 8192;
constexpr int GROUPS = 256;                 // room for the groups' best (128 to 255 of them)
constexpr uint32_t RANKED = 512;            // most keys that are ranked: 8 of 64 threads

__device__ __forceinline__ uint32_t key_of(float f) {
    uint32_t b = __float_as_uint(f);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}

// One compare-exchange stage across the wave: lanes whose bit J is clear keep
// the larger key when `desc`, the smaller otherwise; their partners the other.
template <int J>
__device__ __forceinline__ uint64_t exchange(uint64_t v, uint32_t lane, bool desc) {
    const uint64_t o = gd_lane_xor64<J>(v, lane);
    const bool keep_max = ((lane & J) == 0) == desc;
    return (o > v) == keep_max ? o : v;         // (equal keys: either)
}

// A bitonic sequence (one key per lane) into descending order.
__device__ __forceinline__ uint64_t merge_desc(uint64_t v, uint32_t lane) {
    v = exchange<32>(v, lane, true);
    v = exchange<16>(v, lane, true);
    v = exchange<8>(v, lane, true);
    v = exchange<4>(v, lane, true);
    v = exchange<2>(v, lane, true);
    v = exchange<1>(v, lane, true);
    return v;
}

// Any 64 keys (one per lane) into descending order.
__device__ __forceinline__ uint64_t sort_desc(uint64_t v, uint32_t lane) {
    v = exchange<1>(v, lane, (lane & 2) == 0);
    v = exchange<2>(v, lane, (lane & 4) == 0);
    v = exchange<1>(v, lane, (lane & 4) == 0);
    v = exchange<4>(v, lane, (lane & 8) == 0);
    v = exchange<2>(v, lane, (lane & 8) == 0);
    v = exchange<1>(v, lane, (lane & 8) == 0);
    v = exchange<8>(v, lane, (lane & 16) == 0);
    v = exchange<4>(v, lane, (lane & 16) == 0);
    v = exchange<2>(v, lane, (lane & 16) == 0);
    v = exchange<1>(v, lane, (lane & 16) == 0);
    v = exchange<16>(v, lane, (lane & 32) == 0);
    v = exchange<8>(v, lane, (lane & 32) == 0);
    v = exchange<4>(v, lane, (lane & 32) == 0);
    v = exchange<2>(v, lane, (lane & 32) == 0);
    v = exchange<1>(v, lane, (lane & 32) == 0);
    return merge_desc(v, lane);
}

// 32 bits that never decrease with the key: the count (at most 1 024: 11 bits) and the 21
// leading bits of the middle field that can differ.  A score's are its own; a sum of at most
// 1 024 values of 16 bits stays within +-2^25, so bits 30 .. 26 of the biased sum say nothing.
// (The key's upper half, 16 bits of count and 16 of the middle, is one and the same for all
// sums: every key then reached the threshold and all of them were sorted, 12 us more at 3 230
// nodes.)  Both fields are clamped, so that a digest is monotone whatever the state holds.
__device__ __forceinline__ uint32_t digest_of(const gd_topk_args& a, uint32_t count, uint32_t mid) {
    if (!a.z_last) {
        constexpr uint32_t lo = 0x80000000u - (1u << 25), hi = 0x80000000u + (1u << 25) - 1;
        mid = (min(max(mid, lo), hi) - lo) << 6;
    }
    return min(count, 2047u) << 21 | mid >> 11;
}

// The middle field of a node's key.
__device__ __forceinline__ uint32_t mid_of(const gd_topk_args& a, uint32_t bits) {
    return a.z_last ? key_of(__uint_as_float(bits) + 0.0f)        // -0 ranks as +0
                    : bits ^ 0x80000000u;                         // sum + 2^31: signed order as unsigned
}
__device__ __forceinline__ uint64_t key_from(uint32_t count, uint32_t mid, uint32_t n) {
    return ((uint64_t)count << 48) | ((uint64_t)mid << 16) | (uint64_t)(0xFFFFu - n);
}
__device__ __forceinline__ uint64_t make_key(const gd_topk_args& a, uint32_t n) {
    if (n >= a.N) return 0;                     // padding sorts last (no node's key is 0)
    const uint32_t* mid = a.z_last ? reinterpret_cast<const uint32_t*>(a.z_last)
                                   : reinterpret_cast<const uint32_t*>(a.score_sum);
    return key_from(a.count[n], mid_of(a, mid[n]), n);
}
__device__ __forceinline__ void write_out(const gd_topk_args& a, uint32_t i, uint64_t k) {
    a.idx[i] = (int32_t)(0xFFFFu - (uint32_t)(k & 0xFFFFu));
    if (a.key) a.key[i] = k;
}

// keys[0 .. P), P a power of two, into descending order (all threads of the workgroup).
__device__ __forceinline__ void sort_in_lds(uint64_t* keys, uint32_t P, uint32_t tid) {
    for (uint32_t k = 2; k <= P; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t i = tid; i < P / 2; i += TOPK_NT) {
                const uint32_t lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));   // index with bit j clear
                const uint32_t hi = lo | j;
                const bool desc = (lo & k) == 0;
                const uint64_t x = keys[lo], y = keys[hi];
                if ((x < y) == desc) { keys[lo] = y; keys[hi] = x; }
            }
            __syncthreads();
        }
    }
}

// At most 64 nodes.
__global__ __launch_bounds__(WAVE) void topk_wave_kernel(const gd_topk_args a) {
    const uint32_t lane = threadIdx.x;
    const uint64_t best = sort_desc(make_key(a, lane), lane);
    if (lane < a.k) write_out(a, lane, best);
}

// The a.k largest of keys[0 .. m), m at most CHUNKS * 64, to their places in the output: lane j
// of every wave holds keys j, 64 + j, ..., a wave ranks every sixteenth of them.
template <int CHUNKS>
__device__ __forceinline__ void rank_keys(const gd_topk_args& a, const uint64_t* keys, uint32_t m, uint32_t lane, uint32_t w) {
    constexpr uint32_t WAVES = TOPK_NT / WAVE;
    uint64_t k[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) k[c] = c * WAVE + lane < m ? keys[c * WAVE + lane] : 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
#pragma unroll
        for (uint32_t q = 0; q < WAVE / WAVES; ++q) {
            const uint32_t at = q * WAVES + w;
            if (c * WAVE + at >= m) return;
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k[c], (int)at);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(k[c] >> 32), (int)at);
            const uint64_t x = ((uint64_t)hi << 32) | lo;
            uint32_t r = 0;
#pragma unroll
            for (int d = 0; d < CHUNKS; ++d) r += (uint32_t)__popcll(__ballot(k[d] > x));
            if (r < a.k && lane == 0) write_out(a, r, x);
        }
    }
}

// k <= 64; KPT keys per thread: KPT * TOPK_NT >= N.
template <int KPT>
__global__ __launch_bounds__(TOPK_NT) void topk_short_kernel(const gd_topk_args a) {
    constexpr int ROOM = KPT * TOPK_NT;             // every key may reach the first threshold
    __shared__ uint64_t keys[ROOM];
    __shared__ uint32_t best_of[GROUPS];
    __shared__ uint32_t threshold, n_reach;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), w = __builtin_amdgcn_readfirstlane(tid / WAVE);
    constexpr uint32_t WAVES = TOPK_NT / WAVE;
    // The threads' nodes are neighbours, so that their counts and scores come in one to three
    // loads (both arrays start at multiples of 256 bytes and their room is rounded up to that:
    // the last thread may read past node N - 1, and drops what it read there).
    uint64_t mine[KPT];
    uint32_t digest[KPT], top = 0;
    const uint32_t n0 = tid * KPT;
#pragma unroll
    for (int q = 0; q < KPT; ++q) { mine[q] = 0; digest[q] = 0; }
    if (n0 < a.N) {
        struct alignas(2 * KPT) Counts { uint16_t v[KPT]; };
        struct alignas(4 * KPT > 16 ? 16 : 4 * KPT) Mids { uint32_t v[KPT]; };
        const Counts c = *reinterpret_cast<const Counts*>(a.count + n0);
        const Mids m = a.z_last ? *reinterpret_cast<const Mids*>(a.z_last + n0)
                                : *reinterpret_cast<const Mids*>(a.score_sum + n0);
#pragma unroll
        for (int q = 0; q < KPT; ++q) {
            if (n0 + q < a.N) {
                const uint32_t mid = mid_of(a, m.v[q]);
                mine[q] = key_from(c.v[q], mid, n0 + q);
                digest[q] = digest_of(a, c.v[q], mid);
            }
            top = max(top, digest[q]);
        }
    }
    // groups of g threads, g the largest of 1, 2, 4, 8 that leaves 128 groups with nodes
    const uint32_t used = (a.N + KPT - 1) / KPT;
    const uint32_t lg = used >= 1024 ? 3u : used >= 512 ? 2u : used >= 256 ? 1u : 0u;
    if (lg > 0) top = max(top, gd_lane_xor<1>(top, lane));
    if (lg > 1) top = max(top, gd_lane_xor<2>(top, lane));
    if (lg > 2) top = max(top, gd_lane_xor<4>(top, lane));
    const uint32_t groups = min((used + (1u << lg) - 1) >> lg, (uint32_t)GROUPS);
    if ((tid & ((1u << lg) - 1)) == 0 && (tid >> lg) < (uint32_t)GROUPS) best_of[tid >> lg] = top;
    if (tid == 0) { n_reach = 0; threshold = 0; }
    __syncthreads();
    uint32_t alike = 0;                             // groups whose best reaches the threshold
    if (groups > a.k) {                             // (else every key is ranked)
        // The largest value that at least k values reach.  Lane j holds values j, 64 + j, ...,
        // so a value comes out of a register by its lane number: no LDS round trip in the loop.
        uint32_t v[GROUPS / WAVE], best = 0;
#pragma unroll
        for (int c = 0; c < GROUPS / WAVE; ++c) v[c] = c * WAVE + lane < groups ? best_of[c * WAVE + lane] : 0u;
#pragma unroll
        for (int c = 0; c < GROUPS / WAVE; ++c) {
            if ((uint32_t)c * WAVE >= groups) break;
#pragma unroll
            for (uint32_t q = 0; q < WAVE / WAVES; ++q) {
                const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)v[c], (int)(q * WAVES + w));
                uint32_t reach = 0;
#pragma unroll
                for (int d = 0; d < GROUPS / WAVE; ++d) reach += (uint32_t)__popcll(__ballot(v[d] >= x));
                if (reach >= a.k) best = max(best, x);      // (padding: x = 0 never raises it)
            }
        }
        if (lane == 0) atomicMax(&threshold, best);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < GROUPS / WAVE; ++c) alike += (uint32_t)__popcll(__ballot(v[c] >= threshold));
    }
    const uint32_t thr = threshold;
    uint32_t hits = 0;
    // (many more groups than were asked for: surely more keys than are ranked -- none are gathered)
    const bool crowded = KPT > 1 && alike > a.k + WAVE / 2;
    if (!crowded) {
#pragma unroll
        for (int q = 0; q < KPT; ++q) hits += digest[q] >= thr && mine[q] != 0 ? 1u : 0u;
    }
    if (KPT == 1) {
        // (many threads may hold a hit here, one each: a wave's places in one addition.  1 000 equal
        // scores, k = 64: 8.1 us with an addition a thread, 7.3 so)
        const uint64_t with = __ballot(hits != 0);
        if (with != 0ull) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&n_reach, (uint32_t)__popcll(with));
            base = __builtin_amdgcn_readfirstlane(base);
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(with >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)with, base));
            if (hits) keys[pos] = mine[0];
        }
    } else if (hits) {
        uint32_t pos = atomicAdd(&n_reach, hits);
#pragma unroll
        for (int q = 0; q < KPT; ++q)
            if (digest[q] >= thr && mine[q] != 0) keys[pos++] = mine[q];
    }
    __syncthreads();
    uint32_t m = n_reach;                           // at least min(k, N) = k of them
    if (__builtin_expect(crowded || m > RANKED, 0)) {
        // Digests that are alike throughout.  The k-th largest of the threads' best keys: only
        // the k threads whose best is among those hold keys that reach it, KPT * k at the most.
        // (Threads take every 1 024th node here: equal scores leave the lowest indices, which
        // are neighbours, and one of them per thread is what a threshold of best keys needs.)
        uint64_t best = 0;
#pragma unroll
        for (int q = 0; q < KPT; ++q) mine[q] = make_key(a, q * TOPK_NT + tid);
#pragma unroll
        for (int q = 0; q < KPT; ++q) best = mine[q] > best ? mine[q] : best;
        best = sort_desc(best, lane);
        __syncthreads();                            // (everyone has read the count and is done with the keys)
        keys[tid] = best;
        if (tid == 0) n_reach = 0;
        for (uint32_t half = WAVES / 2; half > 0; half /= 2) {
            // the upper 64 of two sorted lists are a bitonic sequence
            __syncthreads();
            if (w < half) {
                const uint64_t x = keys[w * WAVE + lane], y = keys[(w + half) * WAVE + (WAVE - 1 - lane)];
                keys[w * WAVE + lane] = merge_desc(x > y ? x : y, lane);
            }
        }
        __syncthreads();
        const uint64_t least = keys[a.k - 1];
        __syncthreads();
        hits = 0;
#pragma unroll
        for (int q = 0; q < KPT; ++q) hits += mine[q] >= least && mine[q] != 0 ? 1u : 0u;
        if (hits) {
            uint32_t pos = atomicAdd(&n_reach, hits);
#pragma unroll
            for (int q = 0; q < KPT; ++q)
                if (mine[q] >= least && mine[q] != 0 && pos < RANKED) keys[pos++] = mine[q];
        }
        __syncthreads();
        m = min(n_reach, RANKED);
    }
    if (m <= 2 * WAVE) rank_keys<2>(a, keys, m, lane, w);                  // the usual case
    else if (m <= 4 * WAVE) rank_keys<4>(a, keys, m, lane, w);
    else rank_keys<8>(a, keys, m, lane, w);
}

// Any k: everything sorted.
__global__ __launch_bounds__(TOPK_NT) void topk_sort_kernel(const gd_topk_args a) {
    __shared__ uint64_t keys[TOPK_MAX];
    const uint32_t tid = threadIdx.x;
    uint32_t P = 64;
    while (P < a.N) P <<= 1;                       // power of two >= N, <= TOPK_MAX
    for (uint32_t n = tid; n < P; n += TOPK_NT) keys[n] = make_key(a, n);
    __syncthreads();
    sort_in_lds(keys, P, tid);
    for (uint32_t i = tid; i < a.k; i += TOPK_NT) write_out(a, i, keys[i]);
}

}  // namespace

hipError_t gd_launch_topk(const gd_topk_args& a, hipStream_t s) {
    if (a.k == 0) return hipSuccess;
    if (a.N > TOPK_MAX || a.k > a.N) return hipErrorInvalidValue;
    // (one wave's sort serves up to 64 nodes whatever k is: k <= N)
    if (a.N <= (uint32_t)WAVE) hipLaunchKernelGGL(topk_wave_kernel, dim3(1), dim3(WAVE), 0, s, a);
    else if (a.k > (uint32_t)WAVE) hipLaunchKernelGGL(topk_sort_kernel, dim3(1), dim3(TOPK_NT), 0, s, a);
    else if (a.N <= 1024) hipLaunchKernelGGL(topk_short_kernel<1>, dim3(1), dim3(TOPK_NT), 0, s, a);
    else if (a.N <= 2048) hipLaunchKernelGGL(topk_short_kernel<2>, dim3(1), dim3(TOPK_NT), 0, s, a);
    else if (a.N <= 4096) hipLaunchKernelGGL(topk_short_kernel<4>, dim3(1), dim3(TOPK_NT), 0, s, a);
    else hipLaunchKernelGGL(topk_short_kernel<8>, dim3(1), dim3(TOPK_NT), 0, s, a);
    return hipGetLastError();
}
