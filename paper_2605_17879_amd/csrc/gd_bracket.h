// The bracket of the hinted selection's counting pass and the counter that a value falls into,
// apart from the kernels that use them, so that a host program can go through the bit patterns too.
#ifndef GD_BRACKET_H_
#define GD_BRACKET_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

template <int LOG_NB>
__device__ __forceinline__ int shift_for(uint32_t span) {
    const int width = 32 - __builtin_clz(span | 1u);
    return width > LOG_NB ? width - LOG_NB : 0;            // (span >> shift) < NB
}

// Whether the keys lo .. hi (lo <= hi) can be that bracket: widened to 2^LOG_NB buckets they stay under
// the largest key that is selected by, and a bucket is at least four keys wide.  Narrower ones would
// leave the MAD's edges no room, and, what matters more, a value's bits keep their sign, or a NaN's
// pattern, unless they are shifted by two: the clamp below then holds whatever the column is.  (Counted
// all the same and given up afterwards, columns whose MAD is 5e-5 of their median took, launch: 65 536 ranks
// x 512 x 4 220 us, 201 without; 8 000 x 1 000 x 4 73 and 64; one hinted step of 32 768 x 8 25.0 and 22.0.)
constexpr uint32_t BRACKET_KEY_LIMIT = 0x7D000000u;
template <int LOG_NB>
__device__ __forceinline__ bool bracket_counts(uint32_t lo, uint32_t hi) {
    const uint32_t span = hi - lo;
    return span >= 2u << LOG_NB && span < 0x20000000u && hi < BRACKET_KEY_LIMIT - 2u * span;
}

// Counters: 64 words for what lies under the bracket, the buckets, 64 words for what lies over it;
// a lane has a word of its own on either side.  The bracket starts on a bucket boundary, so that a
// key's bucket is its own bits shifted down, less the bracket's: the clamp works on the shifted bits
// and the subtraction is in the counter's address (three vector instructions a value).
template <int LOG_NB>
struct BracketCounters {
    float cl, ch;              // the shifted bits of the lane's words below and above, as floats
    uint32_t base;             // added to four times the clamped bits: bytes, mod 2^32
    __device__ __forceinline__ BracketCounters(uint32_t first, uint32_t lane) {      // (of the first bucket, shifted down)
        // (below 0, of a bracket that begins at a bucket under 64, `cl` is a NaN, and the median of three is
        // then the least of the others: at least 0, counter 64 - first)
        cl = bits_as_float(first - 1u - lane);
        ch = bits_as_float(first + (1u << LOG_NB) + lane);
        base = (64u - first) * 4u;
    }
    // `shifted` (at most 2^30 - 1) clamped to the two: the median of the three, as floats, whose order
    // theirs is too (positive ones, subnormals among them, and no NaNs).  In bytes, of counters 63 - lane .. 64 + NB + lane.
    template <typename Median>
    __device__ __forceinline__ uint32_t at(uint32_t shifted, uint32_t base_here, Median median) const {
        return (float_as_bits(median(bits_as_float(shifted), cl, ch)) << 2) + base_here;
    }
    static __device__ __forceinline__ float bits_as_float(uint32_t v) { return __builtin_bit_cast(float, v); }
    static __device__ __forceinline__ uint32_t float_as_bits(float v) { return __builtin_bit_cast(uint32_t, v); }
};

#endif  // GD_BRACKET_H_
