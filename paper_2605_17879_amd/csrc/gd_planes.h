// Counting in bit slices: a word holds one bit of each of 32 independent series (32
// ranks or nodes; or the exceed bits of four items' eight metrics), and a count of set
// bits per series is a stack of such words, plane p holding bit p of all 32 counts.
// A full adder on three words is two three-input bit operations (v_bitop3), so adding 64
// steps of 32 series costs about 120 instructions of ONE lane: where every lane has a
// word of its own, a step of a series costs 1/16 of an instruction.
#ifndef GD_PLANES_H_
#define GD_PLANES_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

constexpr int GD_BLOCK_PLANES = 7;     // sums of up to 64 steps
constexpr int GD_COUNT_PLANES = 11;    // sums of up to 1 024 (the longest window) and of 64 more

// a + b + c of every series: sum and carry words
__device__ __forceinline__ void gd_full_add(uint32_t a, uint32_t b, uint32_t c, uint32_t* sum, uint32_t* carry) {
    *sum = a ^ b ^ c;
    *carry = (a & b) | (c & (a | b));
}

// acc += the sixteen words x
__device__ __forceinline__ void gd_add16(uint32_t (&acc)[GD_BLOCK_PLANES], const uint32_t (&x)[16]) {
    uint32_t two[2], four[2], eight[2], c;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int r = 0; r < 2; ++r)
                gd_full_add(acc[0], x[8 * h + 4 * q + 2 * r], x[8 * h + 4 * q + 2 * r + 1], &acc[0], &two[r]);
            gd_full_add(acc[1], two[0], two[1], &acc[1], &four[q]);
        }
        gd_full_add(acc[2], four[0], four[1], &acc[2], &eight[h]);
    }
    gd_full_add(acc[3], eight[0], eight[1], &acc[3], &c);
#pragma unroll
    for (int p = 4; p < GD_BLOCK_PLANES; ++p) {
        const uint32_t t = acc[p] & c;
        acc[p] ^= c;
        c = t;
    }
}

// a += b, a of NA planes and b of NB <= NA
template <int NA, int NB>
__device__ __forceinline__ void gd_planes_add(uint32_t (&a)[NA], const uint32_t (&b)[NB]) {
    static_assert(NB <= NA, "gd_planes_add");
    uint32_t c = 0;
#pragma unroll
    for (int p = 0; p < NA; ++p) {
        if (p < NB) gd_full_add(a[p], b[p], c, &a[p], &c);
        else {
            const uint32_t t = a[p] & c;
            a[p] ^= c;
            c = t;
        }
    }
}

// a -= b (no series of a below b's)
template <int NA, int NB>
__device__ __forceinline__ void gd_planes_sub(uint32_t (&a)[NA], const uint32_t (&b)[NB]) {
    static_assert(NB <= NA, "gd_planes_sub");
    uint32_t borrow = 0;
#pragma unroll
    for (int p = 0; p < NA; ++p) {
        const uint32_t x = a[p], y = p < NB ? b[p] : 0u;
        a[p] = x ^ y ^ borrow;
        borrow = (~x & (y | borrow)) | (y & borrow);
    }
}

// the series whose count has reached K (1 <= K <= 1 024): the carry out of count + (2^NP - K)
template <int NP>
__device__ __forceinline__ uint32_t gd_planes_reach(const uint32_t (&a)[NP], uint32_t K) {
    const uint32_t add = (1u << NP) - K;
    uint32_t c = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t k = (add >> p) & 1u ? 0xFFFFFFFFu : 0u;
        c = (a[p] & k) | (c & (a[p] | k));
    }
    return c;
}

// a + (2^NP - K), one plane more: its last plane says which counts have reached K (1 <= K <= 2^NP).
template <int NP>
__device__ __forceinline__ void gd_planes_bias(const uint32_t (&a)[NP], uint32_t K, uint32_t (&v)[NP + 1]) {
    const uint32_t add = (1u << NP) - K;
    uint32_t c = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) gd_full_add(a[p], (add >> p) & 1u ? 0xFFFFFFFFu : 0u, c, &v[p], &c);
    v[NP] = c;
}

// One step of every series: `in` enters its count, `out` leaves it.  Counting down is counting
// up on the complement, so both are one chain of two instructions a plane.
template <int NP>
__device__ __forceinline__ void gd_planes_step(uint32_t (&v)[NP], uint32_t in, uint32_t out) {
    uint32_t c = in ^ out;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint32_t t = c & (v[p] ^ out);
        v[p] ^= c;
        c = t;
    }
}

// the count of series `bit` in lane `lane`'s planes, for the whole wave
template <int NP>
__device__ __forceinline__ uint32_t gd_planes_count(const uint32_t (&a)[NP], int lane, uint32_t bit) {
    uint32_t c = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p)
        c |= (((uint32_t)__builtin_amdgcn_readlane((int)a[p], lane) >> bit) & 1u) << p;
    return c;
}

#endif  // GD_PLANES_H_
