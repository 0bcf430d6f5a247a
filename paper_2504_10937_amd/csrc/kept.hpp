// Record offsets of the positions of a kept search window (stable-group scan):
// entry i is the end of the records of position lo + i.  They are kept in 32
// bits, half the LDS traffic of the offsets' own 64 (by which the scans of
// 120k and 60k vertices took 0.7-1% longer), for plans whose records they
// count; a plan of triangles holds up to 3 (2^31 - 1) records, and past 2^32
// its offsets are read from P instead.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lds {

// Edge plans always qualify: 2 (2^31 - 1) records (check_edge_count).
inline bool kept_in_32_bits(int64_t records) { return records <= (int64_t)UINT32_MAX; }

__host__ __device__ inline void keep_offset(uint32_t* kept, int64_t i, int64_t end) { kept[i] = (uint32_t)end; }

// P[e + 1], the end of the records of the window's position e
__host__ __device__ inline int64_t kept_end(const uint32_t* kept, bool in_32_bits, int64_t lo, int64_t e,
                                            const int64_t* P) {
    return in_32_bits ? (int64_t)kept[e - lo] : P[e + 1];
}

}  // namespace lds
