// Host checks of the library's own arithmetic at the ends of its ranges, where
// no test input of a usable size reaches: each line that fails is printed, and
// "ok" when none does.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "bucketset.hpp"
#include "chunks.hpp"
#include "graph.hpp"
#include "kept.hpp"
#include "loadcode.hpp"

namespace lds {
void* dev_alloc(size_t, hipStream_t) { return nullptr; }
void dev_free(void*) {}
Graph::~Graph() {}
}  // namespace lds

using namespace lds;

static int failures = 0;
#define EXPECT(cond)                                          \
    do {                                                      \
        if (!(cond)) {                                        \
            std::printf("line %d: %s\n", __LINE__, #cond);    \
            ++failures;                                       \
        }                                                     \
    } while (0)

// a window of 2056 positions with the records of a complete graph's triangles
// (2,110,485 a position, 4,339,157,160 in all), and windows that end at 2^32
static void kept_offsets() {
    const int64_t per = 2055LL * 2054 / 2, n = 2056, lo = 7, top = (int64_t)1 << 32;
    for (int64_t last : {n * per, top - 1, top, top + 1, (int64_t)3 * INT32_MAX}) {
        std::vector<int64_t> P(lo + n + 1, 0);
        std::vector<uint32_t> kept(n);
        for (int64_t i = 0; i < n; ++i) {
            P[lo + i + 1] = last - (n - 1 - i) * (last >= n * per ? per : 1);
            keep_offset(kept.data(), i, P[lo + i + 1]);
        }
        for (int64_t i = 0; i < n; ++i) {
            const int64_t e = lo + i;
            EXPECT(kept_end(kept.data(), kept_in_32_bits(last), lo, e, P.data()) == P[e + 1]);
        }
    }
    EXPECT(kept_in_32_bits(top - 1) && !kept_in_32_bits(top) && kept_in_32_bits(2 * (int64_t)INT32_MAX));
}

// as include/lds.h promises for lds_create_graph
static void edge_count() {
    auto status = [](int64_t m) {
        try {
            check_edge_count(m);
        } catch (const Error& e) {
            return e.code;
        }
        return (int)ST_OK;
    };
    EXPECT(status(0) == ST_OK && status(INT32_MAX) == ST_OK);
    EXPECT(status((int64_t)INT32_MAX + 1) == ST_OVERFLOW && status((int64_t)1 << 33) == ST_OVERFLOW);
}

// 4 items a workgroup of 256 threads (a wave an item) and 16 (16 lanes an item)
static void launches() {
    for (int per : {4, 16})
        for (int64_t items : {(int64_t)0, (int64_t)1, (int64_t)1 << 20, ((int64_t)1 << 26) - 1, (int64_t)1 << 26,
                              (int64_t)1 << 28, (int64_t)INT32_MAX, (int64_t)1 << 33}) {
            const int64_t g = stride_grid(items, per);
            EXPECT(g >= 1 && g * 512 < (int64_t)1 << 32);
            EXPECT(g * per >= items || g == kStrideWG);
        }
}

// codes of loads: monotone, and for the loads about a lone pattern's even split
// (1/h each) told apart to a part in 2^10, at any iteration
static void load_codes() {
    for (int mode : {2, 3, 4}) {
        for (int64_t i : {0, 1, 2, 5, 10, 30, 31, 32, 99, 100, 199, 1000, 20000}) {
            const uint64_t D = fw_denom(mode, i);
            for (int64_t most : {(int64_t)1, (int64_t)65535, (int64_t)65536, (int64_t)INT32_MAX}) {
                const int base = code_base(mode, D), mant = code_mant(most);
                EXPECT(mant == 11 || mant == 12);
                EXPECT(base >= 0 && base < 256 && Codes(base, base, mant).in() == base &&
                       Codes(base, base, mant).mant() == mant);
                int last = -1;
                for (uint64_t A = 0; A <= 64 * D && A < 1000000; A += A < 4096 ? 1 : 1 + A / 5000) {
                    const int c = qcode(A, base, mant);
                    EXPECT(c >= last);
                    last = c;
                }
                // from the even split on (triangles: a tenth below it): a step of 1/1000 apart
                for (int k = mode == 3 ? 900 : 1000; k < 1200; ++k) {
                    const uint64_t a = D * k / (1000 * mode), b = D * (k + 1) / (1000 * mode);
                    if (a >= 64 && (b - a) * 1024 >= b) EXPECT(qcode(b, base, mant) > qcode(a, base, mant));
                }
                // a quarter of the initial load of the vertex of the most patterns is in the window
                const uint64_t A0 = (uint64_t)most * (D / mode) / 4;
                if ((unsigned __int128)most * (D / mode) < ((unsigned __int128)1 << 62))
                    EXPECT(qcode(A0, base, mant) < 65535);
            }
        }
    }
}

// chunks (a multiple of 64 slots, at most kChunk) and pieces fill whole rounds
// of whatever number of waves sweeps them: no more rounds than the largest
// chunks of the size's class need
static void chunk_rounds() {
    for (int64_t waves : {512, 2048, 3072, 4096})
        for (int64_t pieces : {(int64_t)0, waves / 3})
            for (int64_t k : {1, 2, 3, 5}) {
                const int64_t slots = (k * waves - pieces) * kOneBatch - 1;
                const int64_t c = std::min<int64_t>(chunk_slots(slots, pieces, waves) / 64 * 64, kChunk);
                const int64_t rounds = ((slots + c - 1) / c + pieces + waves - 1) / waves;
                EXPECT(c >= kChunkMin && rounds <= k);
            }
}

// the rows of a bucket that share a neighbour, and the neighbours of one row,
// start from places of their own: at least a third as many as the keys
static void bucket_places() {
    for (int vb : {12, 17, 19, 22, 24, 28}) {
        const int rows = 1 << std::min(11, 32 - vb);
        for (uint32_t nb : {0u, 1u, 5u, 1000u, (1u << (vb - 1)) + 3u})
            for (int by_row : {1, 0}) {
                const int n = by_row ? rows : 2048;
                int log2 = 10;
                while ((1 << log2) < 2 * n) ++log2;
                std::vector<char> hit((size_t)1 << log2, 0);
                int places = 0;
                for (int x = 0; x < n; ++x) {
                    const uint32_t key = by_row ? ((uint32_t)x << vb) | (nb & ((1u << vb) - 1)) : ((uint32_t)(rows - 1) << vb) | ((nb + x) & ((1u << vb) - 1));
                    const uint32_t p = bucket_place(key, log2);
                    EXPECT(p < (uint32_t)1 << log2);
                    if (!hit[p]) ++places;
                    hit[p] = 1;
                }
                EXPECT(3 * places >= n);
            }
    }
}

// pieces are whole words, at most kPiece slots, longer in larger plans
static void pieces() {
    for (int64_t waves : {512, 4096}) {
        int last = 0;
        for (int64_t slots : {(int64_t)1100, waves * 128, waves * 128 + 64, kPieceSlots - 1, kPieceSlots, (int64_t)1 << 33}) {
            const int p = piece_slots(slots, slots, waves);
            EXPECT(p % 64 == 0 && p <= kPiece && p >= last);
            EXPECT(piece_slots(slots, 1100, waves) <= p);
            last = p;
        }
    }
}

int main() {
    pieces();
    bucket_places();
    chunk_rounds();
    load_codes();
    launches();
    edge_count();
    kept_offsets();
    if (failures == 0) std::printf("ok\n");
    return failures != 0;
}
