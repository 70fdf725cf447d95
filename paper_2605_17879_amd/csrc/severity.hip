// Severity of the performance impact of the flagged nodes (Section 4.2: the
// tiered response -- no observable impact, a moderate sustained slowdown of
// about 10%, a severe one of 20% or more).
//
// A workgroup looks at up to eight nodes, every gridDim.x-th one: neighbours, which often fall
// behind together (a rack, a switch), are different workgroups' and worked on side by side.  A
// node that is not flagged (its own window count and those of its 8 ranks all below k) reports
// tier 0.  For a flagged node, a few
// dozen of thousands, the workgroup forms the quotient of each of the node's 8
// primary-metric samples of the last min(T, W) steps by that step's cross-rank median and
// takes the median of the at most 8192 quotients minus one.  Missing samples (NaN) are left
// out.
//
// The median is selected, not sorted for: the quotients stay in LDS as order-preserving
// integer keys, the threads count how many lie under two pivots at a time (first around the
// middle of a sorted sample of 64, then where the counts so far put the wanted rank), and
// when at most 64 are left between the pivots they are sorted by one wave's lane exchanges.
// Bound by the length of that chain (loads, divisions, four or five counts, a barrier each).
// Measured (launch, 8 192 nodes, 48 of them flagged, 2 048 quotients each): 42 us with a
// workgroup per node sorting all quotients in LDS (66 stages with a barrier each), 11.8 us.
// Eight neighbours flagged, a call in a row of them: 37 us that way, 10.2 (128 quotients 6.9 and
// 5.5), where one workgroup took the neighbours one after another 48 (17).
#include "gd_internal.h"
#include "gd_lanes.h"

namespace {

constexpr int WAVE = 64;
constexpr int SEV_NT = 512;
constexpr int FEW_NT = 128;       // threads for up to twice as many quotients
constexpr uint32_t GROUP = 8;     // most nodes of a workgroup
constexpr uint32_t GROUPS = 1024; // workgroups: as many as fit the chip at once (four a CU)
constexpr int SEV_MAX = 8192;     // 8 GPUs x the longest window
constexpr uint32_t MISSING = 0xFFFFFFFFu;      // above every key

__device__ __forceinline__ uint32_t key_of(float f) {
    uint32_t b = __float_as_uint(f);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float float_of_key(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

struct Shared {
    uint32_t q[SEV_MAX];
    uint32_t count[2][SEV_NT / WAVE];     // two 16-bit counts of each wave, written in turn
    uint32_t slots[WAVE];         // the last candidates
    uint32_t n_slots, below, above;
};

// Sum over the workgroup of values whose sum fits 32 bits (turn: alternates).
template <int NT>
__device__ __forceinline__ uint32_t block_sum(Shared& sh, uint32_t v, uint32_t turn) {
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    v += gd_lane_xor<1>(v, lane); v += gd_lane_xor<2>(v, lane); v += gd_lane_xor<4>(v, lane);
    v += gd_lane_xor<8>(v, lane); v += gd_lane_xor<16>(v, lane); v += gd_lane_xor<32>(v, lane);
    if (lane == 0) sh.count[turn & 1][threadIdx.x / WAVE] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int w = 0; w < NT / WAVE; ++w) s += sh.count[turn & 1][w];
    return uniform(s);
}

// The order statistics k0 <= k1 <= k0 + 1 of the n keys below MISSING among sh.q[0 .. cnt).
// Throughout, clo keys lie under lo and chi under hi, with clo <= k0 and k1 < chi.  Ends for
// any contents: a round narrows [lo, hi) to a part of it, from the fourth on to a half.
template <int NT>
__device__ __forceinline__ void select(Shared& sh, uint32_t cnt, uint32_t n, uint32_t k0, uint32_t k1, uint32_t turn,
                                       uint32_t* s0, uint32_t* s1) {
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1);
    uint32_t lo = 0, hi = MISSING, clo = 0, chi = n, part = 0;
    // true when one of the pivots p <= q parts the two statistics (k0 < part <= k1)
    auto narrow = [&](uint32_t p, uint32_t q) -> bool {
        uint32_t c = 0;                                    // (at most SEV_MAX in all: no carry between the halves)
        for (uint32_t i = tid; i < cnt; i += NT) {
            const uint32_t k = sh.q[i];
            c += (k < p ? 1u : 0u) + (k < q ? 0x10000u : 0u);
        }
        c = block_sum<NT>(sh, c, turn++);
        bool parted = false;
        auto take = [&](uint32_t at, uint32_t under) {
            const bool up = under <= k0 && at > lo, down = under > k1 && at < hi, splits = under > k0 && under <= k1;
            lo = up ? at : lo; clo = up ? under : clo;
            hi = down ? at : hi; chi = down ? under : chi;
            part = splits ? at : part; parted = parted || splits;
        };
        take(p, c & 0xFFFFu);
        take(q, c >> 16);
        return parted;
    };
    bool parted = false;
    if (n > (uint32_t)WAVE) {
        // around the middle of a sample: two standard deviations of its median's rank
        // (every wave sorts it for itself: no barrier; GPUs in turn)
        const uint32_t sample = sh.q[min(lane * (cnt / WAVE) + (lane & 7), cnt - 1)];
        const uint32_t ns = (uint32_t)__popcll(__ballot(sample < MISSING));
        if (ns >= 16) {
            const uint32_t sorted = gd_sort64(sample), reach = 4u + ns / 16u;
            const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)(ns / 2 - reach));
            const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)sorted, (int)min(ns / 2 + reach, ns - 1)) + 1u;
            parted = narrow(p, q);
        }
        for (int round = 0; !parted && chi - clo > (uint32_t)WAVE; ++round) {
            const uint32_t span = hi - lo;
            if (span <= 1) { *s0 = lo; *s1 = lo; return; }             // ties
            uint32_t p = span / 2, q = p;
            if (round < 3) {
                // the keys between the pivots taken as evenly spread: the wanted rank's place,
                // and 2.5 standard deviations of it to either side
                const float c = (float)(chi - clo), at = (float)(k1 - clo) + 0.5f;
                const float side = 4.0f + 1.25f * __builtin_sqrtf(c), scale = (float)span / c;
                p = (uint32_t)fminf(fmaxf((at - side) * scale, 0.0f), 4294967040.0f);
                q = (uint32_t)fminf(fmaxf((at + side) * scale, 0.0f), 4294967040.0f);
            }
            p = uniform(min(max(p, 1u), span - 1u));
            q = uniform(min(max(q, 1u), span - 1u));
            parted = narrow(lo + p, lo + q);
        }
    }
    if (parted) {
        uint32_t mx = 0, mn = MISSING;
        for (uint32_t i = tid; i < cnt; i += NT) {
            const uint32_t k = sh.q[i];
            if (k < part) mx = max(mx, k);
            else mn = min(mn, k);
        }
        atomicMax(&sh.below, mx);
        atomicMin(&sh.above, mn);
        __syncthreads();
        *s0 = sh.below; *s1 = sh.above;
        return;
    }
    // at most 64 keys in [lo, hi)
    for (uint32_t i = tid; i < cnt; i += NT) {
        const uint32_t k = sh.q[i];
        if (k - lo < hi - lo) {
            const uint32_t to = atomicAdd(&sh.n_slots, 1u);
            if (to < (uint32_t)WAVE) sh.slots[to] = k;
        }
    }
    __syncthreads();
    const uint32_t c = gd_sort64(lane < chi - clo ? sh.slots[lane] : MISSING);
    *s0 = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)((k0 - clo) & (WAVE - 1)));
    *s1 = (uint32_t)__builtin_amdgcn_readlane((int)c, (int)((k1 - clo) & (WAVE - 1)));
}

template <int NT>
__global__ __launch_bounds__(NT) void severity_kernel(const gd_severity_args a) {
    __shared__ Shared sh;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), groups = gridDim.x;
    const uint16_t* rc = reinterpret_cast<const uint16_t*>(a.state + a.lay.rank_count);
    const uint16_t* nc = reinterpret_cast<const uint16_t*>(a.state + a.lay.node_count);
    const uint32_t ws = a.T < a.W ? a.T : a.W, cnt = ws * 8;
    // every wave finds the group's flagged nodes for itself: lane 8 * i + g looks at GPU g of node i
    const uint32_t node = blockIdx.x + (lane / 8) * groups;
    const bool high = node < a.N && (rc[(size_t)node * 8 + (lane & 7)] >= a.K || nc[node] >= a.K);
    const uint64_t flags = ws == 0 ? 0ull : __ballot(high);
    if (tid < WAVE && (lane & 7) == 0 && node < a.N && ((flags >> lane) & 0xFFull) == 0) {
        a.slowdown[node] = 0.0f;
        a.tier[node] = 0;
    }
    for (uint32_t g = 0; g < GROUP; ++g) {
        if (((flags >> (8 * g)) & 0xFFull) == 0) continue;
        const uint32_t n = blockIdx.x + g * groups;
        __syncthreads();                               // (the node before this one is done with the work area)
        if (tid == 0) { sh.n_slots = 0; sh.below = 0; sh.above = MISSING; }
        uint32_t present = 0;
        for (uint32_t i = tid; i < cnt; i += NT) {
            uint32_t k = MISSING;
            const size_t t = a.T - ws + i / 8;
            const float m = a.med[t * a.M + a.primary];
            const float xv = a.x[(t * a.M + a.primary) * (size_t)a.R + (size_t)n * 8 + (i & 7)] + 0.0f;
            float r;
            if (a.dir > 0) r = xv / m;
            else if (a.dir < 0) r = m / xv;
            else r = xv >= m ? xv / m : m / xv;
            // a missing sample (NaN), or a step without a median, is left out
            if (xv == xv && m == m) {
                k = min(key_of(r), MISSING - 1u);
                ++present;
            }
            sh.q[i] = k;
        }
        uint32_t turn = 0;
        const uint32_t np = block_sum<NT>(sh, present, turn++);
        if (np == 0) {                                 // flagged, but nothing arrived inside the window
            if (tid == 0) { a.slowdown[n] = 0.0f; a.tier[n] = 1; }
            continue;
        }
        uint32_t s0, s1;
        select<NT>(sh, cnt, np, (np - 1) / 2, np / 2, turn, &s0, &s1);
        if (tid == 0) {
            // the middle quotient, or the two middle ones added, then halved
            const float mid = (np & 1) ? float_of_key(s1) : 0.5f * (float_of_key(s0) + float_of_key(s1));
            const float s = mid - 1.0f;
            a.slowdown[n] = s;
            a.tier[n] = s >= a.severe ? 3 : (s >= a.moderate ? 2 : 1);
        }
    }
}

}  // namespace

hipError_t gd_launch_severity(const gd_severity_args& a, hipStream_t s) {
    if (a.N == 0) return hipSuccess;
    if (a.N > GROUP * GROUPS) return hipErrorInvalidValue;
    // Few quotients leave most of 512 threads idle, who then only add to the barriers: all of
    // 8 192 nodes flagged, 128 quotients each, 46.7 us with them, 25.0 with 128 (half of them flagged 26.9 and 16.8).
    const dim3 grid(a.N < GROUPS ? a.N : GROUPS);
    if (8 * (a.T < a.W ? a.T : a.W) <= 2 * FEW_NT) hipLaunchKernelGGL(severity_kernel<FEW_NT>, grid, dim3(FEW_NT), 0, s, a);
    else hipLaunchKernelGGL(severity_kernel<SEV_NT>, grid, dim3(SEV_NT), 0, s, a);
    return hipGetLastError();
}
