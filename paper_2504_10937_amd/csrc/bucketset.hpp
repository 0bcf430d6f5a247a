// Where the hash set of a bucket of rows (ingest) looks for a key first.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lds {

// A bucket's key is its row's high bits above the neighbour's id, in 32 bits.
// Multiplicative hashing by the product's top bits, which every bit of the key
// reaches: lower ones miss the row's bits, and the rows that share a neighbour
// (a hub's) then chain from one place (a star's 256 buckets of 1,950 keys took
// 457 us, by the top bits under 20).  log2: of the table's size.
__host__ __device__ inline uint32_t bucket_place(uint32_t key, int log2) { return (key * 2654435769u) >> (32 - log2); }

}  // namespace lds
