// Which ranks the samples of a run's first columns take, apart from the kernel so that a host program can
// tell them too.
#ifndef GD_SAMPLE_H_
#define GD_SAMPLE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

// A wave takes 256 values of one column: four neighbours a lane.  With `waves` in a workgroup up to four share
// a column: 2 to the power of this.
__device__ __forceinline__ uint32_t sample_parts_log(uint32_t columns, uint32_t waves) {
    return 4u * columns <= waves ? 2u : 2u * columns <= waves ? 1u : 0u;
}
// The first of the four ranks of lane `place` mod 64 of the column's part `place` / 64.  Sixteen neighbours
// at a time (64 bytes) are spread over the ranks by multiples of the golden ratio, a step that no
// structure of the job shares.
__device__ __forceinline__ uint32_t sample_rank(uint32_t place, uint32_t R) {
    const uint32_t piece = (uint32_t)((uint64_t)(place / 4u * 0x9E3779B9u) * (R / 16u) >> 32);
    const uint32_t from = piece * 16u + (place & 3u) * 4u;
    return from < R - 4u ? from : R - 4u;
}

#endif  // GD_SAMPLE_H_
