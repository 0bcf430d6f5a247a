// Sizes of the chunks and hub-row pieces into which a sweep plan cuts the rows
// (see graph.hpp).
#pragma once
#include <algorithm>
#include <cstdint>

namespace lds {

// Target slots of a chunk for a plan with `slots` slots outside the hub rows
// and `pieces` hub pieces, swept by `waves` waves (sweep_waves).  A sweep runs
// in rounds (every wave takes one chunk or piece), so the size is the smallest
// that fills a whole number of rounds.  A round costs a chain of dependent
// reads, then a batch of 256 slots (512 from 2^22 slots on) at a time: up to
// kOneBatch slots (with the part of the last row that a chunk takes beyond its
// target) is the best size while there are few rounds, kTwoBatches once there
// are many, and tiny plans use kChunkMin, to have more waves in flight.
// Measured per sweep in us on 4096 waves, by size: 37M slots 1024 236, 960 221,
// 384 236; 4.4M 1024 44, 768 35, 384 33, 256 40; 2.9M 512 18.9, 384 17.2, 256
// 20.2; 1.6M 512 17.0, 384 15.5, 256 20.5; 24k 512 8.1, 256 6.8, 128 5.9, 64 6.4.
constexpr int kChunkMin = 128;
constexpr int kOneBatch = 448;
constexpr int kTwoBatches = 960;
inline int64_t chunk_slots(int64_t slots, int64_t pieces, int64_t waves) {
    if (slots <= waves * kChunkMin) return kChunkMin;
    const int64_t per = slots <= 3 * waves * kOneBatch ? kOneBatch : kTwoBatches;
    const int64_t rounds = (slots / per + pieces + waves - 1) / waves;
    const int64_t chunks = std::max<int64_t>(1, rounds * waves - pieces);
    return std::max<int64_t>(kChunkMin, (slots + chunks - 1) / chunks + 63);
}

// Most slots of a hub-row piece.  A piece is one wave's, so a plan under
// kPieceSlots cuts shorter ones; but each adds its wins to its row's counter,
// and many pieces of few rows queue there: past a quarter of the waves they are
// twice as long.  us a sweep by 512 and 1024: 20 rows of 100,000 slots 35.2 and
// 23.6, 500 of 2000 11.0 and 8.7, 4-cliques of K_64 26.4 and 17.3, triangles of
// K_150 10.6 and 10.8, of 20k vertices with 32 hub rows 8.0 and 8.1.
constexpr int64_t kPieceSlots = (int64_t)1 << 22;
inline int piece_slots(int64_t slots, int64_t hub_slots, int64_t waves) {
    if (slots >= kPieceSlots) return 2048;
    return hub_slots > waves / 4 * 512 ? 1024 : 512;
}

}  // namespace lds
