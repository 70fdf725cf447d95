// Cross-lane helpers shared by the kernels: wave-wide moves with immediate
// patterns (DPP, swizzle, permlane swap) -- no address registers involved.
#ifndef GD_LANES_H_
#define GD_LANES_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

// Value held by lane (lane ^ J) of the same wave, J a power of two below 64.  No exchange
// goes through the LDS crossbar (ds_swizzle): a sort of 64 keys by one wave is a chain of
// 21 of them, and a crossbar round trip costs about ten times a DPP move.
template <int J>
__device__ __forceinline__ uint32_t gd_lane_xor(uint32_t v, uint32_t lane) {
    if constexpr (J == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
    else if constexpr (J == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
    else if constexpr (J == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);
    else if constexpr (J == 4) {       // mirrored within 8 lanes (i ^ 7), then within 4 (i ^ 3)
        const int m = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, true);
    } else if constexpr (J == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane & 16) ? r[0] : r[1];
    }
    else {
        static_assert(J == 32, "gd_lane_xor");
        auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane & 32) ? r[0] : r[1];
    }
}

template <int J>
__device__ __forceinline__ uint64_t gd_lane_xor64(uint64_t v, uint32_t lane) {
    const uint32_t lo = gd_lane_xor<J>((uint32_t)v, lane);
    const uint32_t hi = gd_lane_xor<J>((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Which lanes keep the smaller key in the stage of distance J that merges runs of S: a
// constant, so that it is a scalar literal and no lane works it out (nor keeps it in
// registers from one sort to the next).
template <int J, int S>
constexpr uint64_t gd_keeps_smaller() {
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l)
        if (((l & J) == 0) == ((l & S) == 0)) m |= 1ull << l;
    return m;
}
template <int BIT>
constexpr uint64_t gd_lanes_with() {
    uint64_t m = 0;
    for (int l = 0; l < 64; ++l)
        if (l & BIT) m |= 1ull << l;
    return m;
}

// The lanes of a constant mask.  INLOOP: made where it is used, from words that the optimiser
// cannot see through -- in a kernel that sorts inside a loop it would otherwise keep all of a
// sort's masks in scalar registers across the loop, and spill them.
template <uint64_t MASK, bool INLOOP>
__device__ __forceinline__ bool gd_lane_in() {
    if constexpr (!INLOOP) return __builtin_amdgcn_inverse_ballot_w64(MASK);
    uint32_t lo = (uint32_t)MASK, hi = (uint32_t)(MASK >> 32);
    asm volatile("" : "+s"(lo), "+s"(hi));
    return __builtin_amdgcn_inverse_ballot_w64((uint64_t)hi << 32 | lo);
}

// One compare-exchange stage across the wave.
template <int J, int S, bool INLOOP>
__device__ __forceinline__ uint32_t gd_exchange(uint32_t v) {
    uint32_t o;
    if constexpr (J == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        o = gd_lane_in<gd_lanes_with<16>(), INLOOP>() ? r[0] : r[1];
    } else if constexpr (J == 32) {
        auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        o = gd_lane_in<gd_lanes_with<32>(), INLOOP>() ? r[0] : r[1];
    } else {
        o = gd_lane_xor<J>(v, 0);
    }
    return gd_lane_in<gd_keeps_smaller<J, S>(), INLOOP>() ? min(v, o) : max(v, o);
}
template <int S, bool INLOOP>
__device__ __forceinline__ uint32_t gd_merge(uint32_t v) {
    if constexpr (S > 32) v = gd_exchange<32, S, INLOOP>(v);
    if constexpr (S > 16) v = gd_exchange<16, S, INLOOP>(v);
    if constexpr (S > 8) v = gd_exchange<8, S, INLOOP>(v);
    if constexpr (S > 4) v = gd_exchange<4, S, INLOOP>(v);
    if constexpr (S > 2) v = gd_exchange<2, S, INLOOP>(v);
    return gd_exchange<1, S, INLOOP>(v);
}

// 64 keys, one per lane, into ascending order.
template <bool INLOOP = false>
__device__ __forceinline__ uint32_t gd_sort64(uint32_t v) {
    v = gd_merge<2, INLOOP>(v);
    v = gd_merge<4, INLOOP>(v);
    v = gd_merge<8, INLOOP>(v);
    v = gd_merge<16, INLOOP>(v);
    v = gd_merge<32, INLOOP>(v);
    return gd_merge<64, INLOOP>(v);
}

// Transpose of the 64x64 bit matrix whose row i is the word held by lane i:
// afterwards bit j of lane i is what bit i of lane j was.  For every index bit
// K the rows and columns exchange that bit (a butterfly with the lane i ^ K).
template <int K>
__device__ __forceinline__ uint64_t gd_transpose_stage(uint64_t x, uint32_t lane) {
    constexpr uint64_t m = K == 32 ? 0x00000000FFFFFFFFull
                         : K == 16 ? 0x0000FFFF0000FFFFull
                         : K == 8  ? 0x00FF00FF00FF00FFull
                         : K == 4  ? 0x0F0F0F0F0F0F0F0Full
                         : K == 2  ? 0x3333333333333333ull
                                   : 0x5555555555555555ull;
    const uint64_t p = gd_lane_xor64<K>(x, lane);
    if ((lane & K) == 0) {
        const uint64_t t = ((x >> K) ^ p) & m;
        return x ^ (t << K);
    }
    const uint64_t t = ((p >> K) ^ x) & m;
    return x ^ t;
}

__device__ __forceinline__ uint64_t gd_transpose64(uint64_t x, uint32_t lane) {
    x = gd_transpose_stage<32>(x, lane);
    x = gd_transpose_stage<16>(x, lane);
    x = gd_transpose_stage<8>(x, lane);
    x = gd_transpose_stage<4>(x, lane);
    x = gd_transpose_stage<2>(x, lane);
    x = gd_transpose_stage<1>(x, lane);
    return x;
}

#endif  // GD_LANES_H_
