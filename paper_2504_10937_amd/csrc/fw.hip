// Frank-Wolfe iterations of Alg. 1 (edges, Eq. cp) and Alg. 6 (triangles,
// Eq. trcp) on gfx950, in exact integer form, and the same iteration over
// 4-cliques (the h-clique program that Eq. trcp generalises, h = 4).
//
// State.  With gamma_i = 2/(i+2) every load is r_u^(i) = A_u / D_i with the
// common denominator D_i = (i+1)(i+2) (edges), 3(i+1)(i+2) (triangles) or
// 2(i+1)(i+2) (4-cliques), and the update r <- (1-gamma) r + gamma b becomes
// A_u += inc_i * b_u with inc_i = D_i - D_{i-1} = 2(i+1), 6(i+1) or 4(i+1),
// b_u = units won in iteration i.  Each vertex carries one packed 64-bit key
//     K_u = (A_u << B) | (2^B - 1 - orig_id(u)),
// so "smallest load, ties to the larger original id" is a single unsigned
// compare, and adding (inc * b) << B updates A without touching the id bits.
//
// Sweep (one launch per iteration, keys ping-pong between two buffers so that
// every decision reads r^(i-1)).  Pull over incidence slots: a vertex wins a
// slot's pattern iff its key is below the keys of the other h-1 vertices.
//   * chunk waves: a wave64 streams one row-aligned chunk in 64-slot words, a
//     batch of words in flight; the wave ballot of wins is a word's decision
//     word of the iteration (stored once, coalesced); then a lane per row
//     counts its slots' wins in the chunk's words with popcounts (no atomics)
//     and writes the row's new key and code.
//   * hub pieces: a row with more slots than a chunk is cut into word-aligned
//     pieces, one wave each, dealt over all waves with the chunks; a piece
//     adds its wins to the row's counter and the wave that completes the row's
//     last piece writes the row's key.
// The duality-gap terms sum_u A_u^2 and sum_u A_u b_u (= sum over patterns of
// the winning numerator, i.e. the minimum) are accumulated exactly in 128-bit
// integers per workgroup and reduced once after the last iteration.
#include "batch.hpp"
#include "graph.hpp"
#include "loadcode.hpp"
#include "push.hpp"
#include "wave.hpp"

#include <mutex>
#include <type_traits>

// Scratch of lds_frank_wolfe_noalloc, for callers that cannot allocate device
// memory: the per-workgroup gap partial sums of every iteration, their
// per-iteration totals and the gap values.  One copy per device (4 MiB),
// held until the process ends; host code reaches it only through the
// address hipGetSymbolAddress returns for the current device.
static constexpr size_t kScratchWords = (size_t)1 << 19;
static __device__ __align__(256) uint64_t scratch[kScratchWords];

namespace lds {

namespace {

typedef unsigned __int128 u128;

struct SweepArgs {
    const int32_t* rid;
    const int64_t* rp;
    const int32_t* py;
    int64_t n_hub;
    const int64_t* hwo;
    int64_t n_pieces;
    int piece;           // most slots of a piece
    const int32_t* hp_row;
    const int32_t* hp_off;
    unsigned long long* hub_ctr;  // per hub row: (pieces done << 40) | wins so far
    int64_t n_chunks;
    const ChunkDesc* desc;
    const uint64_t* head;
    int64_t chunk_words;
    const uint64_t* Kin;
    uint64_t* Kout;
    const uint16_t* Qin;  // 16-bit codes of the loads (see qcode)
    uint16_t* Qout;
    Codes codes;         // of Qin (D_(i-1)) and Qout (D_i)
    uint64_t* bits;      // this iteration's decision words
    uint64_t inc;
    int B;
    uint64_t* partial;   // 4 words per workgroup (or nullptr)
    int ncache;          // codes staged in LDS: min(n, kCacheQ)
    // 2D part (edge plans of large graphs; n_parts = 0 otherwise)
    int64_t n_parts;
    const int32_t* part_blk;
    const int32_t* part_j0;
    const int32_t* part_j1;
    const int64_t* part_lo;
    const int64_t* part_hi;
    const int64_t* hseg;
    const int64_t* hblk_row;
    const uint32_t* hpay;
    uint32_t* part_cnt;
    int64_t hP;
    int hR, hC;
    int64_t n_heavy;
    int64_t hword0;
    int64_t nv;          // vertices (slabs are clipped to it)
    // hub push (n_push > 0; edge plans only): the pieces above are those of
    // the hub prefixes, hub_pre[r] slots of hub row r; every workgroup stores
    // its hub counters (pstride words, two 16-bit counts each) at
    // push_part + blockIdx * pstride
    int64_t n_push;
    const int32_t* hub_pre;
    uint32_t* push_part;
    int64_t pstride;
};

__device__ inline uint64_t readlane64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// the h-1 other vertices of the pattern stored at a slot; the slot arrays
// are streamed once per iteration, so they are read non-temporally to keep
// the caches for the gathered keys.  PK: packed (4-cliques), kept packed until
// a member is used
template <int H, bool PK>
struct Slot {
    int32_t v[H - 1];
    static constexpr int kWords = H - 1;
    __device__ inline uint32_t id(int q) const { return (uint32_t)v[q]; }
};
template <>
struct Slot<4, true> {
    uint64_t x;
    static constexpr int kWords = 2;
    __device__ inline uint32_t id(int q) const { return (uint32_t)PackedSlot::id(x, q); }
};

template <int H, bool PK>
__device__ inline Slot<H, PK> load_slot(const int32_t* __restrict__ py, int64_t s);
template <>
__device__ inline Slot<2, false> load_slot<2, false>(const int32_t* __restrict__ py, int64_t s) {
    Slot<2, false> r;
    r.v[0] = __builtin_nontemporal_load(py + s);
    return r;
}
template <>
__device__ inline Slot<3, false> load_slot<3, false>(const int32_t* __restrict__ py, int64_t s) {
    const long long x = __builtin_nontemporal_load(reinterpret_cast<const long long*>(py) + s);
    Slot<3, false> r;
    r.v[0] = (int32_t)(uint32_t)(unsigned long long)x;
    r.v[1] = (int32_t)(uint32_t)((unsigned long long)x >> 32);
    return r;
}
template <>
__device__ inline Slot<4, false> load_slot<4, false>(const int32_t* __restrict__ py, int64_t s) {
    Slot<4, false> r;
    r.v[0] = __builtin_nontemporal_load(py + 3 * s);
    r.v[1] = __builtin_nontemporal_load(py + 3 * s + 1);
    r.v[2] = __builtin_nontemporal_load(py + 3 * s + 2);
    return r;
}
template <>
__device__ inline Slot<4, true> load_slot<4, true>(const int32_t* __restrict__ py, int64_t s) {
    Slot<4, true> r;
    r.x = (uint64_t)__builtin_nontemporal_load(reinterpret_cast<const long long*>(py) + s);
    return r;
}

#ifndef LDS_SWEEP_THREADS
#define LDS_SWEEP_THREADS 1024
#endif
#ifndef LDS_SWEEP_CACHE
#define LDS_SWEEP_CACHE 77824
#endif
#ifndef LDS_SWEEP_WG_PER_CU
#define LDS_SWEEP_WG_PER_CU 1
#endif
// 64-slot words of a chunk or piece in flight per wave.  A batch costs its
// instructions whether its words are there or not, and a chunk of a small plan
// has few: 4 words up to kWideSlots slots (24k slots 7.0 -> 5.8 us a sweep, 2.9M
// 17.9 -> 17.2; triangles 84k 8.5 -> 7.8, 1.6M 16.2 -> 15.3), 8 above (4.8M slots
// 32 us, 34 with 4; 206M 823 and 837; triangles 37M 213 and 218).
constexpr int kWordsSmall = 4, kWordsLarge = 8;
constexpr int64_t kWideSlots = (int64_t)1 << 22;
constexpr int kPT = LDS_SWEEP_THREADS;      // threads of a persistent workgroup
constexpr int kWaves = kPT / 64;
constexpr int kCacheQ = LDS_SWEEP_CACHE;    // codes of the first (highest-degree) vertices staged in LDS
constexpr int kWgPerCU = LDS_SWEEP_WG_PER_CU;

// code of vertex v: from the LDS copy for the hot prefix, else from memory
__device__ inline uint16_t qload(const uint16_t* __restrict__ qc, int nc, const uint16_t* __restrict__ Q,
                                 uint32_t v) {
    uint16_t q;
    if (v < (uint32_t)nc)
        q = qc[v];
    else
        q = Q[v];
    return q;
}

// Decisions of G slots per lane: does the row vertex (code qu[j], key ku(j))
// beat the other members of the pattern at slot sl[j]?  The members' codes are
// gathered one member at a time, the last one first (members are stored by
// internal id, descending, so the last has the smallest id, the most slots and
// most often a code in LDS): a slot that has lost needs no further gathers.
// Equal codes are settled by the 64-bit keys after every code has been
// compared, all reads of a few slots in flight together: ties are 0.1-2% of
// the slots, but most batches hold one, and a read and wait per tied word was
// the longest part of a batch's chain of dependent reads.
template <int H, int G, bool PK, class KU>
__device__ inline void decide(const uint16_t* __restrict__ qc, int nc, const uint16_t* __restrict__ Q,
                              const uint64_t* __restrict__ K, const Slot<H, PK> (&sl)[G], const bool (&in)[G],
                              const uint16_t (&qu)[G], KU ku, bool (&win)[G]) {
    // Triangles and 4-cliques, whose first member has the largest id: a batch
    // with every code in LDS reads them all without masks and compares once
    // with the smallest (the sweep of 195M clique slots, 20,000 hub rows among
    // 41,000: 504 -> 404 us; half of its cycles went into the masked gathers,
    // 51 vector instructions a word).  Members of a slot that is not lower than
    // the smallest code have larger keys, so a tie is settled by all of them.
    if (H > 2) {
        uint32_t top = 0;
#pragma unroll
        for (int j = 0; j < G; ++j) top = max(top, sl[j].id(0));
        if (__ballot(top >= (uint32_t)nc) == 0) {
            uint16_t q[G][H - 1];
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int x = 0; x < H - 1; ++x) q[j][x] = qc[sl[j].id(x)];
            bool tie[G], any = false;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                uint32_t m = q[j][0];
#pragma unroll
                for (int x = 1; x < H - 1; ++x) m = min(m, (uint32_t)q[j][x]);
                win[j] = in[j] && qu[j] <= m;
                tie[j] = in[j] && qu[j] == m;
                any = any || tie[j];
            }
            if (__ballot(any) == 0) return;
            constexpr int S = G % 4 == 0 ? 4 : G % 3 == 0 ? 3 : G;
#pragma unroll
            for (int j0 = 0; j0 < G; j0 += S) {
                uint64_t k0[S], kv[S][H - 1];
#pragma unroll
                for (int j = 0; j < S; ++j) {
                    k0[j] = 0;
#pragma unroll
                    for (int x = 0; x < H - 1; ++x) kv[j][x] = ~0ull;
                    if (tie[j0 + j]) {
                        k0[j] = ku(j0 + j);
#pragma unroll
                        for (int x = 0; x < H - 1; ++x) kv[j][x] = K[sl[j0 + j].id(x)];
                    }
                }
#pragma unroll
                for (int j = 0; j < S; ++j)
#pragma unroll
                    for (int x = 0; x < H - 1; ++x) win[j0 + j] = win[j0 + j] && k0[j] < kv[j][x];
            }
            return;
        }
    }
    uint32_t tied[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        win[j] = in[j];
        tied[j] = 0;
    }
#pragma unroll
    for (int q = H - 2; q >= 0; --q) {
        uint16_t qv[G];
#pragma unroll
        for (int j = 0; j < G; ++j) qv[j] = win[j] ? qload(qc, nc, Q, sl[j].id(q)) : (uint16_t)0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
            if (qu[j] == qv[j]) tied[j] |= 1u << q;
            win[j] = win[j] && qu[j] <= qv[j];
        }
    }
    constexpr int S = H == 2 ? G : (G % 4 == 0 ? 4 : G % 3 == 0 ? 3 : G);  // slots whose keys are in flight together
#pragma unroll
    for (int j0 = 0; j0 < G; j0 += S) {
        uint64_t k0[S], kv[S][H - 1];
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int x = j0 + j;
            k0[j] = 0;
#pragma unroll
            for (int q = 0; q < H - 1; ++q) kv[j][q] = ~0ull;
            if (win[x] && tied[x]) {
                k0[j] = ku(x);
#pragma unroll
                for (int q = 0; q < H - 1; ++q)
                    if (H == 2 || ((tied[x] >> q) & 1u)) kv[j][q] = K[sl[x].id(q)];
            }
        }
#pragma unroll
        for (int j = 0; j < S; ++j)
#pragma unroll
            for (int q = 0; q < H - 1; ++q) win[j0 + j] = win[j0 + j] && k0[j] < kv[j][q];
    }
}

// LDS bytes of the 2D part: block codes (u16) and win counts (u32), two slabs
constexpr size_t kHeavyLds = (size_t)kHeavyRows * 2 + (size_t)kHeavyRows * 4 + (size_t)2 * kHeavySlab * 2;
constexpr int kSlabChunks = (kHeavySlab / 8 + kPT - 1) / kPT;  // 16-byte chunks of a slab per thread

// slab j's codes, 16 bytes (8 codes) per chunk, clipped to the vertex count
__device__ inline void slab_load(const uint16_t* __restrict__ Q, int64_t nv, int64_t first, int C, uint4 (&st)[kSlabChunks]) {
#pragma unroll
    for (int q = 0; q < kSlabChunks; ++q) {
        const int c = (int)threadIdx.x + kPT * q;
        const int64_t v = first + 8 * (int64_t)c;
        uint4 x = make_uint4(0, 0, 0, 0);
        if (8 * c < C) {
            if (v + 8 <= nv) {
                x = *reinterpret_cast<const uint4*>(Q + v);
            } else {
                uint16_t e[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) e[k] = (v + k < nv) ? Q[v + k] : (uint16_t)0;
                x.x = e[0] | ((uint32_t)e[1] << 16);
                x.y = e[2] | ((uint32_t)e[3] << 16);
                x.z = e[4] | ((uint32_t)e[5] << 16);
                x.w = e[6] | ((uint32_t)e[7] << 16);
            }
        }
        st[q] = x;
    }
}

__device__ inline void slab_store(uint16_t* __restrict__ slab, int C, const uint4 (&st)[kSlabChunks]) {
#pragma unroll
    for (int q = 0; q < kSlabChunks; ++q) {
        const int c = (int)threadIdx.x + kPT * q;
        if (8 * c < C) reinterpret_cast<uint4*>(slab)[c] = st[q];
    }
}

// The 2D part of an edge sweep (heavy rows; see HeavyPlan).  A workgroup
// takes whole parts.  It stages the block's codes and zeroed win counts in
// LDS, then walks the part's slabs: slab j's codes sit in one LDS buffer
// while the next slab's are loaded into registers and stored into the other
// buffer; the segment's words are decided with both codes from LDS (64-bit
// keys only on equal codes), each word's ballot is its decision word, and
// the wins of each run of one row within a word are added to the row's LDS
// count once.  The part's counts go to part_cnt; k_heavy_finish sums the
// parts of each row after the sweep.
template <bool ENABLE>
__device__ inline void heavy_parts(const SweepArgs& a, uint8_t* dyn, int64_t* sgc) {
    if constexpr (ENABLE) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const int R = a.hR, C = a.hC;
        uint16_t* rq = reinterpret_cast<uint16_t*>(dyn);
        uint32_t* rc = reinterpret_cast<uint32_t*>(dyn + (size_t)kHeavyRows * 2);
        uint16_t* slabs = reinterpret_cast<uint16_t*>(dyn + (size_t)kHeavyRows * 6);
        const uint64_t le = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
        for (int64_t pt = blockIdx.x; pt < a.n_parts; pt += gridDim.x) {
            const int64_t b = a.part_blk[pt];
            const int64_t j0 = a.part_j0[pt], j1 = a.part_j1[pt];
            const int64_t lo = a.part_lo[pt], hi = a.part_hi[pt];
            const int64_t row0 = a.hblk_row[b];
            const int nr = (int)(a.hblk_row[b + 1] - row0);
            // the part's segment bounds, clipped to its positions, staged in
            // LDS when they fit (a few hundred slabs)
            const int64_t* sgg = a.hseg + b * a.hP;
            const bool cached = j1 - j0 + 1 <= kWaves * 32;
            for (int64_t k = threadIdx.x; cached && k <= j1 - j0; k += kPT) sgc[k] = min(max(sgg[j0 + k], lo), hi);
            for (int i = threadIdx.x; i < nr; i += kPT) {
                rq[i] = a.Qin[row0 + i];
                rc[i] = 0u;
            }
            __syncthreads();
            auto bound = [&](int64_t j) { return cached ? sgc[j - j0] : min(max(sgg[j], lo), hi); };
            auto next_j = [&](int64_t j) {
                while (j < j1 && bound(j + 1) <= bound(j)) ++j;
                return j;
            };
            int64_t j = next_j(j0);
            uint4 st[kSlabChunks];
            if (j < j1) {
                slab_load(a.Qin, a.nv, j * C, C, st);
                slab_store(slabs, C, st);
            }
            __syncthreads();
            int cur = 0;
            while (j < j1) {
                const int64_t jn = next_j(j + 1);
                if (jn < j1) slab_load(a.Qin, a.nv, jn * C, C, st);
                const uint16_t* sl = slabs + (size_t)cur * kHeavySlab;
                const int64_t q0 = bound(j), q1 = bound(j + 1);
                const uint64_t* __restrict__ Kin = a.Kin;
                constexpr int U = 8;
                for (int64_t base = q0 + (int64_t)64 * U * w; base < q1; base += (int64_t)64 * U * kWaves) {
                    uint32_t x[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int64_t pos = base + 64 * u + lane;
                        x[u] = pos < q1 ? __builtin_nontemporal_load(a.hpay + pos) : 0xffffffffu;
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool valid = x[u] != 0xffffffffu;
                        const uint32_t rl = (x[u] >> 16) & 0x7fffu, nl = x[u] & 0xffffu;
                        bool win = false;
                        if (valid) {
                            const uint16_t qu = rq[rl], qv = sl[nl];
                            win = (qu != qv) ? (qu < qv) : (Kin[row0 + rl] < Kin[j * C + nl]);
                        }
                        const uint64_t W = __ballot(win);
                        const int64_t wpos = base + 64 * u;
                        if (lane == 0 && wpos < q1) __builtin_nontemporal_store(W, a.bits + a.hword0 + wpos / 64);
                        // runs of one row within the word (run heads are marked
                        // in the payload): one LDS add per run
                        const uint64_t V = __ballot(valid);
                        const uint64_t Hm = __ballot(valid && (x[u] >> 31));
                        const uint64_t nv1 = (V >> lane) >> 1, nh1 = (Hm >> lane) >> 1;  // next lane's bits (0 past 63)
                        const bool last = valid && (!(nv1 & 1ull) || (nh1 & 1ull));
                        if (last) {
                            const uint64_t hm = Hm & le;
                            const uint64_t from = hm ? (~0ull << (63 - __clzll(hm))) : ~0ull;
                            const uint32_t c = (uint32_t)__popcll(W & le & from);
                            if (c) atomicAdd(&rc[rl], c);
                        }
                    }
                }
                if (jn < j1) slab_store(slabs + (size_t)(cur ^ 1) * kHeavySlab, C, st);
                __syncthreads();
                cur ^= 1;
                j = jn;
            }
            for (int i = threadIdx.x; i < nr; i += kPT) a.part_cnt[pt * R + i] = rc[i];
            __syncthreads();
        }
    }
}

// Persistent sweep: one workgroup per CU.  The workgroup first copies the
// codes of the kCacheQ highest-degree vertices (internal ids [0, kCacheQ))
// into LDS; those vertices take most of the gathers of a power-law graph.
// It then processes hub pieces and chunks, one wave each, dealt over the
// waves of the grid, kG words at a time.  HEAVY: with the 2D part.
template <int H, bool HEAVY, bool GAP, bool PK, int kG>
__global__ __launch_bounds__(kPT) void k_fw_sweep(SweepArgs a) {
    constexpr bool IDENT = H == 2;  // compact row = vertex
    extern __shared__ __align__(16) uint16_t qc[];
    __shared__ uint64_t red[kWaves][4];
    __shared__ uint64_t words[kWaves][32];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nc = a.ncache;
    // in a vector register: the scalar ones are full, and another of them cost a
    // plan of 3M slots 17.2 -> 18.9 us in spills
    Codes codes = a.codes;
    asm("" : "+v"(codes.x));
    // the 2D part first (its LDS layout), then the hot codes for the rest
    heavy_parts<HEAVY>(a, reinterpret_cast<uint8_t*>(qc), reinterpret_cast<int64_t*>(&words[0][0]));
    // Triangles: the wave's first chunk is read before the codes are staged, so
    // that its chain of reads (descriptor; payload, row vertices, keys) runs
    // behind the staging, and the hub pieces come last (24k slots 7.8 -> 6.9 us
    // a sweep, 84k 10.0 -> 9.1, 1.6M 16.1 -> 15.3).  Edges, whose rows need one
    // read less, lost by the registers it holds (3M slots 17.7 -> 18.5, 206M
    // 822 -> 841), and 4-cliques spill.
    constexpr bool kAhead = H == 3;
    // Pieces and chunks are dealt to the waves in turn (the chunks from the wave
    // after the last piece's on), so no wave has two more than another.
    // Neighbouring chunks (rows with cached codes in common) go to the waves of
    // one workgroup, except in a plan that leaves waves without work, which is
    // dealt over the compute units first.
    const bool few = a.n_pieces + a.n_chunks <= (int64_t)gridDim.x * kWaves;
    const int64_t cstep = (int64_t)gridDim.x * kWaves;
    int64_t c0 = few ? (int64_t)w * gridDim.x + blockIdx.x : (int64_t)blockIdx.x * kWaves + w;
    c0 -= a.n_pieces % cstep;
    if (c0 < 0) c0 += cstep;
    ChunkDesc d{}, dn{};
    if (c0 < a.n_chunks) d = a.desc[c0];
    if (kAhead && c0 + cstep < a.n_chunks) dn = a.desc[c0 + cstep];
    // row-start flags of the chunk's words (lane t: word t), bounds, vertex and
    // key of its first 64 rows (lane l: row l), and its first batch's payload
    uint64_t hreg, pk;
    int pa, pb;
    uint32_t pu;
    Slot<H, PK> sl[kG];
    constexpr int PW = Slot<H, PK>::kWords;
    auto load_batch = [&](int t0) {
#pragma unroll
        for (int j = 0; j < kG; ++j) {
            const int off = (t0 + j) * 64 + lane;
            if (H > 2 || off < d.nsl) sl[j] = load_slot<H, PK>(a.py + d.s0 * PW, H > 2 ? min(off, d.nsl - 1) : off);
        }
    };
    auto load_chunk = [&]() {
        if (d.nrows <= 0) return;
        if (kAhead) load_batch(0);
        hreg = (lane < ((d.nsl + 63) >> 6)) ? __builtin_nontemporal_load(a.head + d.w0 + lane) : 0ull;
        const int64_t rl = (int64_t)d.r0 + min(lane, d.nrows - 1);
        pa = (int)(a.rp[rl] - d.s0);
        pb = (int)(a.rp[rl + 1] - d.s0);
        pu = IDENT ? (uint32_t)rl : (uint32_t)a.rid[rl];
        pk = a.Kin[pu];
    };
    if (kAhead) load_chunk();
    // the hot codes, 16 bytes per load and all of a thread's loads in flight
    // (2-byte loads took 10 of the 28 us of a 3M-slot sweep)
    {
        const uint4* __restrict__ src = reinterpret_cast<const uint4*>(a.Qin);
        const int n16 = nc >> 3;
#pragma unroll 4
        for (int i = threadIdx.x; i < n16; i += kPT) reinterpret_cast<uint4*>(qc)[i] = src[i];
        for (int i = (n16 << 3) + threadIdx.x; i < nc; i += kPT) qc[i] = a.Qin[i];
    }
    // hub push: the hub rows' win counters of this workgroup, after the codes
    const int Hp = H == 2 && !HEAVY ? (int)a.n_push : 0;
    uint32_t* hcnt = reinterpret_cast<uint32_t*>(qc + ((nc + 1) & ~1));
    for (int i = threadIdx.x; i < (Hp + 1) / 2; i += kPT) hcnt[i] = 0u;
    __syncthreads();
    u128 sq = 0, mn = 0;
    // ---- hub rows: cut into word-aligned pieces of <= kPiece slots, one wave
    //      each.  A piece stores its decision words and adds (1 << 40) + its
    //      wins to the row's counter with one atomic, so the wave whose add
    //      completes the row's last piece reads the row's total from the value
    //      returned, with no fence; it writes the row's key and clears the
    //      counter for the next sweep.  With the hub push a piece covers only
    //      the row's hub prefix and adds its wins alone: k_push_finish adds
    //      the pushed wins and writes the key.
    auto sweep_pieces = [&]() {
        for (int64_t pc = few ? (int64_t)w * gridDim.x + blockIdx.x : (int64_t)blockIdx.x * kWaves + w; pc < a.n_pieces;
             pc += (int64_t)gridDim.x * kWaves) {
            const int64_t r = a.hp_row[pc];
            const uint32_t u = IDENT ? (uint32_t)r : (uint32_t)a.rid[r];
            const int64_t rs = a.rp[r], re = a.rp[r + 1];
            const int64_t s0 = rs + a.hp_off[pc];
            // offsets within the piece in 32 bits
            const int len = (int)min((Hp > 0 ? rs + a.hub_pre[r] : re) - s0, (int64_t)a.piece);
            const int32_t* __restrict__ pyc = a.py + s0 * PW;
            const uint64_t Ku = a.Kin[u];
            const uint16_t Qu = qcode(Ku >> a.B, codes.in(), codes.mant());
            uint64_t* bw = a.bits + a.chunk_words + a.hwo[r] + (s0 - rs) / 64;
            uint32_t cnt = 0;
            for (int base = 0; base < len; base += 64 * kG) {
                Slot<H, PK> sl[kG];
                bool in[kG], win[kG];
                uint16_t qu[kG];
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    const int off = base + 64 * j + lane;
                    in[j] = off < len;
                    if (H > 2 || in[j]) sl[j] = load_slot<H, PK>(pyc, H > 2 ? min(off, len - 1) : off);
                    qu[j] = Qu;
                }
                decide<H, kG, PK>(qc, nc, a.Qin, a.Kin, sl, in, qu, [&](int) { return Ku; }, win);
                uint64_t mine = 0;
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    const uint64_t W = __ballot(win[j]);
                    if (lane == j) mine = W;
                    cnt += (uint32_t)__popcll(W);
                }
                if (lane < kG && base + 64 * lane < len) __builtin_nontemporal_store(mine, bw + base / 64 + lane);
            }
            if (lane == 0 && Hp > 0) {
                atomicAdd(a.hub_ctr + r, (unsigned long long)cnt);
            } else if (lane == 0) {
                const unsigned long long npc = (unsigned long long)((re - rs + a.piece - 1) / a.piece);
                const unsigned long long old = atomicAdd(a.hub_ctr + r, (1ull << 40) | (unsigned long long)cnt);
                if ((old >> 40) == npc - 1) {
                    const uint64_t tot = (old & ((1ull << 40) - 1)) + cnt;
                    const uint64_t Kn = Ku + ((tot * a.inc) << a.B);
                    a.Kout[u] = Kn;
                    a.Qout[u] = qcode(Kn >> a.B, codes.out(), codes.mant());
                    if (GAP) {
                        const uint64_t A = Ku >> a.B;
                        sq += (u128)A * A;
                        mn += (u128)A * tot;
                    }
                    atomicExch(a.hub_ctr + r, 0ull);
                }
            }
        }
    };
    if (!kAhead) sweep_pieces();
    // ---- chunks: one wave each
    //   A. decision words: kG words per batch, slot payloads then codes in
    //      flight; each word's ballot is kept by lane t
    //   B. one lane per row: popcount of the row's slot range in the chunk's
    //      decision words (staged in LDS), key and code update
    // A wave's time is a chain of dependent reads, so what does not depend on
    // the decisions is read ahead: the next chunk's descriptor during this
    // chunk (two ahead with kAhead), and the bounds and keys of the first 64 rows before the first
    // batch (their codes also serve the slots of chunks of at most 64 rows).
    ChunkDesc dnn{};
    for (int64_t c = c0; c < a.n_chunks; c += cstep, d = kAhead ? dn : dnn, dn = dnn) {
        dnn = ChunkDesc{};
        constexpr int kDescAhead = kAhead ? 2 : 1;
        if (c + kDescAhead * cstep < a.n_chunks) dnn = a.desc[c + kDescAhead * cstep];
        if (!kAhead || c != c0) load_chunk();
        const int nrows = d.nrows;
        if (nrows <= 0) continue;
        const int64_t r0 = d.r0, s0 = d.s0, w0 = d.w0;
        const int nsl = d.nsl, nw = (nsl + 63) >> 6;  // <= 32: a chunk spans < 2048 slots
        const uint64_t le = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
        const int pq = (int)qcode(pk >> a.B, codes.in(), codes.mant());
        const bool small = nrows <= 64;
        int32_t rowrel = -1;  // chunk-relative row of the slot before the current word
        uint64_t mybits = 0;
        for (int t0 = 0; t0 < nw; t0 += kG) {
            if (!kAhead || t0 > 0) load_batch(t0);
            uint64_t Hw[kG];
#pragma unroll
            for (int j = 0; j < kG; ++j) Hw[j] = readlane64(hreg, t0 + j);  // t0 + j < 40
            int32_t row[kG];
            bool val[kG];
            int32_t rb = rowrel;
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                const int off = (t0 + j) * 64 + lane;
                val[j] = off < nsl;
                row[j] = rb + (int32_t)__popcll(Hw[j] & le);
                rb += (int32_t)__popcll(Hw[j]);
            }
            rowrel = rb;
            uint16_t qu[kG];
            if (small) {
#pragma unroll
                for (int j = 0; j < kG; ++j) qu[j] = (uint16_t)__shfl(pq, row[j], 64);
            } else {
#pragma unroll
                for (int j = 0; j < kG; ++j)
                    qu[j] = val[j] ? qload(qc, nc, a.Qin,
                                           IDENT ? (uint32_t)(r0 + row[j]) : (uint32_t)a.rid[r0 + row[j]])
                                   : (uint16_t)0;
            }
            bool win[kG];
            decide<H, kG, PK>(qc, nc, a.Qin, a.Kin, sl, val, qu,
                          [&](int j) { return a.Kin[IDENT ? (uint32_t)(r0 + row[j]) : (uint32_t)a.rid[r0 + row[j]]]; },
                          win);
#pragma unroll
            for (int j = 0; j < kG; ++j) {
                if (H == 2 && Hp > 0 && val[j] && !win[j]) {  // a hub's win, pushed to its counter
                    const uint32_t v = sl[j].id(0);
                    if (v < (uint32_t)Hp) atomicAdd(&hcnt[v >> 1], 1u << ((v & 1u) * 16));
                }
                const uint64_t W = __ballot(win[j]);
                if (lane == t0 + j) mybits = W;
            }
        }
        if (lane < nw) {
            __builtin_nontemporal_store(mybits, a.bits + w0 + lane);
            words[w][lane] = mybits;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int rbase = 0; rbase < nrows; rbase += 64) {
            const int sa = pa, sb = pb;  // sb > sa
            const uint32_t u = pu;
            const uint64_t Ku = pk;
            if (rbase + 64 < nrows) {  // the next 64 rows
                const int64_t rn = r0 + min(rbase + 64 + lane, nrows - 1);
                pa = (int)(a.rp[rn] - s0);
                pb = (int)(a.rp[rn + 1] - s0);
                pu = IDENT ? (uint32_t)rn : (uint32_t)a.rid[rn];
                pk = a.Kin[pu];
            }
            if (rbase + lane < nrows) {
                uint32_t cnt = 0;
                for (int wd = sa >> 6; wd <= ((sb - 1) >> 6); ++wd) {
                    const int lo = max(sa - wd * 64, 0), hi = min(sb - wd * 64, 64);
                    const uint64_t mk = ((hi >= 64) ? ~0ull : ((1ull << hi) - 1ull)) & (~0ull << lo);
                    cnt += (uint32_t)__popcll(words[w][wd] & mk);
                }
                const uint64_t Kn = Ku + (((uint64_t)cnt * a.inc) << a.B);
                a.Kout[u] = Kn;
                a.Qout[u] = qcode(Kn >> a.B, codes.out(), codes.mant());
                if (GAP) {
                    const uint64_t A = Ku >> a.B;
                    sq += (u128)A * A;
                    mn += (u128)A * cnt;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();  // words[w] is rewritten by the next chunk
    }
    if (kAhead) sweep_pieces();
    if (Hp > 0) {  // this workgroup's hub counters (uniform branch)
        __syncthreads();
        uint32_t* o = a.push_part + (int64_t)blockIdx.x * a.pstride;
        for (int i = threadIdx.x; i < (Hp + 1) / 2; i += kPT) o[i] = hcnt[i];
    }
    if (GAP) {
        sq = wave::sum128_lane63(sq);
        mn = wave::sum128_lane63(mn);
        if (lane == 63) {
            red[w][0] = (uint64_t)sq;
            red[w][1] = (uint64_t)(sq >> 64);
            red[w][2] = (uint64_t)mn;
            red[w][3] = (uint64_t)(mn >> 64);
        }
        __syncthreads();
        if (w == 0) {
            u128 S = 0, M = 0;
            if (lane < kWaves) {
                S = ((u128)red[lane][1] << 64) | red[lane][0];
                M = ((u128)red[lane][3] << 64) | red[lane][2];
            }
            S = wave::sum128_lane63(S);
            M = wave::sum128_lane63(M);
            if (lane == 63) {
                uint64_t* o = a.partial + (int64_t)blockIdx.x * 4;
                o[0] = (uint64_t)S;
                o[1] = (uint64_t)(S >> 64);
                o[2] = (uint64_t)M;
                o[3] = (uint64_t)(M >> 64);
            }
        }
    }
}

// per iteration: sum the per-workgroup partials exactly
__global__ __launch_bounds__(256) void k_gap_reduce(const uint64_t* partial, int64_t nblocks, uint64_t* out) {
    __shared__ uint64_t red[4][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t* p = partial + (int64_t)blockIdx.x * nblocks * 4;
    u128 S = 0, M = 0;
    for (int64_t b = threadIdx.x; b < nblocks; b += 256) {
        S += ((u128)p[4 * b + 1] << 64) | p[4 * b];
        M += ((u128)p[4 * b + 3] << 64) | p[4 * b + 2];
    }
    S = wave::sum128_lane63(S);
    M = wave::sum128_lane63(M);
    if (lane == 63) {
        red[w][0] = (uint64_t)S;
        red[w][1] = (uint64_t)(S >> 64);
        red[w][2] = (uint64_t)M;
        red[w][3] = (uint64_t)(M >> 64);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        S = 0;
        M = 0;
        for (int q = 0; q < 4; ++q) {
            S += ((u128)red[q][1] << 64) | red[q][0];
            M += ((u128)red[q][3] << 64) | red[q][2];
        }
        out[4 * blockIdx.x + 0] = (uint64_t)S;
        out[4 * blockIdx.x + 1] = (uint64_t)(S >> 64);
        out[4 * blockIdx.x + 2] = (uint64_t)M;
        out[4 * blockIdx.x + 3] = (uint64_t)(M >> 64);
    }
}

// After a sweep with the hub push: hub row r's wins are its prefix's wins
// (hub_ctr, cleared here for the next sweep) plus the counts every sweep
// workgroup pushed (the r & 1 half of word r >> 1 of its slice); then the
// row's new key and code, and its gap terms (per workgroup, written after
// the sweep's own partial sums of the iteration).  A workgroup takes 64 hub
// rows, one per lane; its four waves each sum every fourth sweep
// workgroup's counts (16 loads in flight per lane), and wave 0 finishes.
template <bool GAP>
__global__ __launch_bounds__(256) void k_push_finish(unsigned long long* hub_ctr, const uint32_t* push_part,
                                                     int64_t pstride, int nblocks, int64_t n_push,
                                                     const uint64_t* Kin, uint64_t* Kout, uint16_t* Qout,
                                                     uint64_t inc, int B, Codes codes, uint64_t* partial) {
    __shared__ uint64_t ps[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t r = (int64_t)blockIdx.x * 64 + lane;
    uint64_t part = 0;
    if (r < n_push) {
        const uint32_t* col = push_part + (r >> 1);
        const int sh = (int)(r & 1) * 16;
#pragma unroll 16
        for (int b = w; b < nblocks; b += 4) part += (col[(int64_t)b * pstride] >> sh) & 0xffffu;
    }
    ps[w][lane] = part;
    __syncthreads();
    if (w != 0) return;
    u128 sq = 0, mn = 0;
    if (r < n_push) {
        const uint64_t tot = hub_ctr[r] + ps[0][lane] + ps[1][lane] + ps[2][lane] + ps[3][lane];
        hub_ctr[r] = 0ull;
        const uint64_t Ku = Kin[r];
        const uint64_t Kn = Ku + ((tot * inc) << B);
        Kout[r] = Kn;
        Qout[r] = qcode(Kn >> B, codes.out(), codes.mant());
        if (GAP) {
            const uint64_t A = Ku >> B;
            sq = (u128)A * A;
            mn = (u128)A * tot;
        }
    }
    if (GAP) {  // wave 0 alone: all 64 lanes active
        sq = wave::sum128_lane63(sq);
        mn = wave::sum128_lane63(mn);
        if (lane == 63) {
            uint64_t* o = partial + (int64_t)blockIdx.x * 4;
            o[0] = (uint64_t)sq;
            o[1] = (uint64_t)(sq >> 64);
            o[2] = (uint64_t)mn;
            o[3] = (uint64_t)(mn >> 64);
        }
    }
}

// After a sweep with a 2D part: every heavy row's wins summed over the parts
// of its block, its new key and code, and the gap terms of those rows (per
// workgroup, written after the sweep's own partial sums of the iteration).
template <bool GAP>
__global__ __launch_bounds__(256) void k_heavy_finish(const uint32_t* part_cnt, const int32_t* blk_part,
                                                      const int32_t* row_blk, const int64_t* blk_row, int R,
                                                      int64_t n_heavy, const uint64_t* Kin, uint64_t* Kout,
                                                      uint16_t* Qout, uint64_t inc, int B, Codes codes, uint64_t* partial) {
    __shared__ uint64_t red[4][4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    u128 sq = 0, mn = 0;
    for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < n_heavy; r += (int64_t)gridDim.x * 256) {
        const int64_t b = row_blk[r], rl = r - blk_row[b];
        const int p0 = blk_part[b], p1 = blk_part[b + 1];
        uint64_t tot = 0;
        int p = p0;
        for (; p + 8 <= p1; p += 8) {
            uint32_t c[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) c[k] = part_cnt[(int64_t)(p + k) * R + rl];
#pragma unroll
            for (int k = 0; k < 8; ++k) tot += c[k];
        }
        for (; p < p1; ++p) tot += part_cnt[(int64_t)p * R + rl];
        const uint64_t Ku = Kin[r];
        const uint64_t Kn = Ku + ((tot * inc) << B);
        Kout[r] = Kn;
        Qout[r] = qcode(Kn >> B, codes.out(), codes.mant());
        if (GAP) {
            const uint64_t A = Ku >> B;
            sq += (u128)A * A;
            mn += (u128)A * tot;
        }
    }
    if (GAP) {
        sq = wave::sum128_lane63(sq);
        mn = wave::sum128_lane63(mn);
        if (lane == 63) {
            red[w][0] = (uint64_t)sq;
            red[w][1] = (uint64_t)(sq >> 64);
            red[w][2] = (uint64_t)mn;
            red[w][3] = (uint64_t)(mn >> 64);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            u128 S = 0, M = 0;
            for (int q = 0; q < 4; ++q) {
                S += ((u128)red[q][1] << 64) | red[q][0];
                M += ((u128)red[q][3] << 64) | red[q][2];
            }
            uint64_t* o = partial + (int64_t)blockIdx.x * 4;
            o[0] = (uint64_t)S;
            o[1] = (uint64_t)(S >> 64);
            o[2] = (uint64_t)M;
            o[3] = (uint64_t)(M >> 64);
        }
    }
}

// initial keys: A0 = deg (edges, r0 = deg/2 with D0 = 2), 2 t_u (triangles,
// r0 = t_u/3 with D0 = 6) or q_u (4-cliques, r0 = q_u/4 with D0 = 4), packed
// with the original-id code
__global__ void k_init_keys(const int32_t* count, int mult, const int32_t* orig_of, int64_t n, int B,
                            uint64_t* K0, uint64_t* K1, Codes codes, uint16_t* Q0, uint16_t* Q1) {
    const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (u >= n) return;
    const uint64_t idm = (1ull << B) - 1ull;
    const uint64_t A = (uint64_t)count[u] * (uint64_t)mult;
    const uint64_t k = (A << B) | (idm - (uint64_t)orig_of[u]);
    K0[u] = k;
    K1[u] = k;
    Q0[u] = Q1[u] = qcode(A, codes.in(), codes.mant());
}

__global__ void k_loads(const uint64_t* K, const int32_t* orig_of, int64_t n, int B, double D, float* r32,
                        uint64_t* A_out) {
    const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (u >= n) return;
    const uint64_t A = K[u] >> B;
    const int32_t o = orig_of[u];
    if (r32) r32[o] = (float)((double)A / D);
    if (A_out) A_out[o] = A;
}

// exact split numerator of every incidence slot from the stored decision
// words: a = a0 + sum_i inc_i [slot won in iteration i], inc_i = incm (i+1)
template <int H, bool PK>
__global__ void k_splits(const int64_t* rp, const int32_t* rid, const int32_t* py, const int64_t* bitbase,
                         int64_t nrows, int64_t nslots, const uint64_t* bits, int64_t total_words, int iters,
                         uint64_t a0, uint64_t incm, const int32_t* orig_of, int32_t* verts, uint64_t* num) {
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= nslots) return;
    // row of slot s: last r with rp[r] <= s
    int64_t lo = 0, hi = nrows - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (rp[mid] <= s) lo = mid; else hi = mid - 1;
    }
    const int64_t r = lo;
    if (bitbase[r] < 0) return;  // a heavy row: k_splits_heavy
    const int64_t pos = bitbase[r] + (s - rp[r]);
    uint64_t a = a0;
    for (int i = 1; i <= iters; ++i) {
        const uint64_t wd = bits[(int64_t)(i - 1) * total_words + pos / 64];
        if ((wd >> (pos % 64)) & 1ull) a += incm * (uint64_t)(i + 1);
    }
    const int32_t x = rid ? rid[r] : (int32_t)r;
    verts[H * s] = orig_of[x];
    const Slot<H, PK> sl = load_slot<H, PK>(py, s);
    for (int j = 0; j < H - 1; ++j) verts[H * s + 1 + j] = orig_of[sl.id(j)];
    num[s] = a;
}

// the same for the slots of heavy rows (edges), position by position of the
// 2D part: the slot is csr[pos], its decision bits follow from word0
__global__ void k_splits_heavy(const uint32_t* csr, const uint32_t* pay, int64_t positions, int64_t word0,
                               const int64_t* rp, int64_t nrows, const int32_t* py, const uint64_t* bits,
                               int64_t total_words, int iters, uint64_t a0, uint64_t incm, const int32_t* orig_of,
                               int32_t* verts, uint64_t* num) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= positions || pay[k] == 0xffffffffu) return;
    const int64_t s = csr[k];
    int64_t lo = 0, hi = nrows - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (rp[mid] <= s) lo = mid; else hi = mid - 1;
    }
    uint64_t a = a0;
    const int64_t pos = word0 * 64 + k;
    for (int i = 1; i <= iters; ++i) {
        const uint64_t wd = bits[(int64_t)(i - 1) * total_words + pos / 64];
        if ((wd >> (pos % 64)) & 1ull) a += incm * (uint64_t)(i + 1);
    }
    verts[2 * s] = orig_of[lo];
    verts[2 * s + 1] = orig_of[py[s]];
    num[s] = a;
}

uint64_t denom(int mode, int64_t i) { return fw_denom(mode, i); }

// the codes of iteration i's sweep (i = 0: of the initial loads)
Codes codes_of(const Graph& g, int mode, int64_t i) {
    const int64_t most = mode == 2 ? g.max_deg : mode == 3 ? g.t_max : g.q_max;
    return Codes(code_base(mode, denom(mode, i > 0 ? i - 1 : 0)), code_base(mode, denom(mode, i)), code_mant(most));
}

template <int H, bool HEAVY, bool PK, int W>
void launch_sweep(const SweepArgs& a, unsigned blocks, bool gap, hipStream_t s) {
    const size_t push_lds = a.n_push > 0 ? (size_t)((a.ncache + 1) & ~1) * 2 + (size_t)a.pstride * 4 : 0;
    const size_t lds = std::max(std::max((size_t)a.ncache * sizeof(uint16_t), push_lds), HEAVY ? kHeavyLds : (size_t)0);
    const int max_lds = (int)std::max((size_t)kCacheQ * 2 + 16, HEAVY ? kHeavyLds : (size_t)0);
    if (gap) {
        static bool attr = false;
        if (!attr) {
            LDS_HIP(hipFuncSetAttribute((const void*)k_fw_sweep<H, HEAVY, true, PK, W>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, max_lds));
            attr = true;
        }
        k_fw_sweep<H, HEAVY, true, PK, W><<<blocks, kPT, lds, s>>>(a);
    } else {
        static bool attr = false;
        if (!attr) {
            LDS_HIP(hipFuncSetAttribute((const void*)k_fw_sweep<H, HEAVY, false, PK, W>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, max_lds));
            attr = true;
        }
        k_fw_sweep<H, HEAVY, false, PK, W><<<blocks, kPT, lds, s>>>(a);
    }
}

// one persistent workgroup per compute unit
unsigned sweep_grid() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        LDS_HIP(hipGetDevice(&dev));
        LDS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        if (cus <= 0) cus = 1;
    }
    return (unsigned)(cus * kWgPerCU);
}

}  // namespace

int64_t sweep_waves() { return (int64_t)sweep_grid() * kWaves; }

namespace {

// workgroups that have a chunk, piece or part to sweep (at least one)
unsigned sweep_blocks(const SweepPlan& p) {
    const int64_t work = p.n_chunks + (p.n_push > 0 ? p.n_ppieces : p.n_pieces) + p.heavy.n_parts;
    return (unsigned)std::min<int64_t>(sweep_grid(), std::max<int64_t>(1, work));
}

// workgroups of the heavy rows' finishing kernel (0 without a 2D part); its
// gap partial sums follow the sweep's in each iteration's slice
unsigned finish_grid(const SweepPlan& p) { return p.heavy.n_parts > 0 ? sweep_grid() : 0u; }

// workgroups of the hub push's finishing kernel (64 hub rows each); its gap
// partial sums follow the sweep's likewise (a plan has a 2D part or the push,
// never both)
unsigned push_grid(const SweepPlan& p) { return (unsigned)((p.n_push + 63) / 64); }

// switch the sweep arguments to the hub push of plan p (sweep workgroups
// `blocks`; push_part sized here)
void use_push(const SweepPlan& p, FwState& f, unsigned blocks, SweepArgs& a, hipStream_t s) {
    a.n_push = p.n_push;
    a.hub_pre = p.hub_pre.p;
    a.n_pieces = p.n_ppieces;
    a.hp_row = p.pp_row.p;
    a.hp_off = p.pp_off.p;
    a.ncache = (int)p.push_nc;
    a.pstride = (p.n_push + 1) / 2;
    const size_t words = (size_t)blocks * (size_t)a.pstride;
    if (f.push_part.n < words) f.push_part.alloc(words, s);
    a.push_part = f.push_part.p;
}

void fill_sweep_args(const Graph& g, const SweepPlan& p, SweepArgs& a) {
    a = SweepArgs{};
    a.rid = p.rid;
    a.rp = p.rp;
    a.py = p.py;
    a.n_hub = p.n_hub;
    a.hwo = p.hwo.p;
    a.n_pieces = p.n_pieces;
    a.piece = p.piece;
    a.hp_row = p.hp_row.p;
    a.hp_off = p.hp_off.p;
    a.hub_ctr = p.hub_ctr.p;
    a.n_chunks = p.n_chunks;
    a.desc = p.desc.p;
    a.head = p.head.p;
    a.chunk_words = p.chunk_words;
    a.B = g.idbits;
    a.ncache = (int)std::min<int64_t>(g.n, kCacheQ);
    const HeavyPlan& h = p.heavy;
    a.n_parts = h.n_parts;
    a.part_blk = h.part_blk.p;
    a.part_j0 = h.part_j0.p;
    a.part_j1 = h.part_j1.p;
    a.part_lo = h.part_lo.p;
    a.part_hi = h.part_hi.p;
    a.hseg = h.seg.p;
    a.hblk_row = h.blk_row.p;
    a.hpay = h.pay.p;
    a.part_cnt = h.part_cnt.p;
    a.hP = h.P;
    a.hR = h.R;
    a.hC = h.C;
    a.n_heavy = h.n_heavy;
    a.hword0 = h.word0;
    a.nv = g.n;
}

// iteration i: the sweep, then the heavy rows' keys; partial = this
// iteration's gap slice (sweep workgroups, then finishing workgroups) or null
void sweep_iteration(const Graph& g, FwState& f, const SweepPlan& p, SweepArgs& a, int mode, int i, unsigned blocks,
                     uint64_t* partial, hipStream_t s) {
    const bool gap = partial != nullptr;
    a.Kin = f.K[f.cur].p;
    a.Kout = f.K[f.cur ^ 1].p;
    a.Qin = f.Q[f.cur].p;
    a.Qout = f.Q[f.cur ^ 1].p;
    a.bits = f.bits.p + (size_t)(i - 1) * p.total_words;
    a.inc = denom(mode, i) - denom(mode, i - 1);
    a.codes = codes_of(g, mode, i);
    a.partial = partial;
    auto launch = [&](auto words) {
        constexpr int W = decltype(words)::value;
        if (mode == 2)
            launch_sweep<2, false, false, W>(a, blocks, gap, s);
        else if (mode == 3)
            launch_sweep<3, false, false, W>(a, blocks, gap, s);
        else if (p.packed)
            launch_sweep<4, false, true, W>(a, blocks, gap, s);
        else
            launch_sweep<4, false, false, kWordsLarge>(a, blocks, gap, s);
    };
    if (a.n_parts > 0)
        launch_sweep<2, true, false, kWordsLarge>(a, blocks, gap, s);
    else if (p.nslots < kWideSlots)
        launch(std::integral_constant<int, kWordsSmall>{});
    else
        launch(std::integral_constant<int, kWordsLarge>{});
    LDS_HIP(hipGetLastError());
    if (a.n_push > 0) {
        const unsigned pg = push_grid(p);
        if (gap)
            k_push_finish<true><<<pg, 256, 0, s>>>(a.hub_ctr, a.push_part, a.pstride, (int)blocks, a.n_push, a.Kin,
                                                   a.Kout, a.Qout, a.inc, a.B, a.codes, partial + (size_t)blocks * 4);
        else
            k_push_finish<false><<<pg, 256, 0, s>>>(a.hub_ctr, a.push_part, a.pstride, (int)blocks, a.n_push,
                                                    a.Kin, a.Kout, a.Qout, a.inc, a.B, a.codes, nullptr);
        LDS_HIP(hipGetLastError());
    }
    const unsigned fb = finish_grid(p);
    if (fb > 0) {
        const HeavyPlan& h = p.heavy;
        uint64_t* fp = gap ? partial + (size_t)blocks * 4 : nullptr;
        if (gap)
            k_heavy_finish<true><<<fb, 256, 0, s>>>(h.part_cnt.p, h.blk_part.p, h.row_blk.p, h.blk_row.p, h.R,
                                                    h.n_heavy, a.Kin, a.Kout, a.Qout, a.inc, a.B, a.codes, fp);
        else
            k_heavy_finish<false><<<fb, 256, 0, s>>>(h.part_cnt.p, h.blk_part.p, h.row_blk.p, h.blk_row.p, h.R,
                                                     h.n_heavy, a.Kin, a.Kout, a.Qout, a.inc, a.B, a.codes, fp);
        LDS_HIP(hipGetLastError());
    }
    f.cur ^= 1;
}

}  // namespace

unsigned __int128 fw_max_numerator(const Graph& g, int mode, int iters) {
    // a vertex that wins every incident pattern in every iteration:
    // deg (1 + sum_i 2(i+1)), t (2 + sum_i 6(i+1)) or q (1 + sum_i 4(i+1))
    const unsigned __int128 N = (unsigned)iters;
    if (mode == 2) return (unsigned __int128)(uint64_t)g.max_deg * (N * N + 3 * N + 1);
    if (mode == 3) return (unsigned __int128)(uint64_t)g.t_max * (2 + 3 * N * (N + 3));
    return (unsigned __int128)(uint64_t)g.q_max * (1 + 2 * N * (N + 3));
}

void fw_prepare(Graph& g, int mode, int iters, hipStream_t s) {
    LDS_CHECK(mode >= 2 && mode <= 4, ST_INVALID, "mode must be LDS_EDGE, LDS_TRIANGLE or LDS_CLIQUE4");
    LDS_CHECK(iters >= 0, ST_INVALID, "iters must be >= 0");
    if (mode == 3 && g.T < 0) list_triangles(g, s);
    if (mode == 4 && g.Q4 < 0) list_cliques4(g, s);
    const SweepPlan& p = plan_of(g, mode);
    FwState& f = g.fw[mode_slot(mode)];
    const int B = g.idbits;
    // overflow: the largest numerator must leave B bits for the id code
    const u128 amax = fw_max_numerator(g, mode, iters);
    LDS_CHECK(B < 64 && (amax >> (64 - B)) == 0, ST_OVERFLOW, "exact load numerator would overflow the 64-bit key");
    const int64_t n = g.n;
    if (f.K[0].n != (size_t)n) {
        f.K[0].alloc(n, s);
        f.K[1].alloc(n, s);
        f.Q[0].alloc(n, s);
        f.Q[1].alloc(n, s);
    }
    const size_t nbits = (size_t)iters * (size_t)p.total_words;
    if (f.bits.n < nbits) f.bits.alloc(nbits, s);
}

void fw_gap_from_sums(FwState& f, int mode, int iters, const uint64_t* sums) {
    f.gap.assign(iters, 0.0);
    f.lb.assign(iters, 0.0);
    f.fval.assign(iters, 0.0);
    for (int i = 1; i <= iters; ++i) {
        const u128 S = ((u128)sums[4 * (i - 1) + 1] << 64) | sums[4 * (i - 1)];
        const u128 M = ((u128)sums[4 * (i - 1) + 3] << 64) | sums[4 * (i - 1) + 2];
        const uint64_t D = denom(mode, i - 1);
        // (D^2/2) gap = sum A^2 - D * sum_patterns min A  (exact)
        const u128 num = S - (u128)D * M;
        const long double LD = (long double)D;
        const long double gap = 2.0L * (long double)num / (LD * LD);
        f.gap[i - 1] = (double)gap;
        f.lb[i - 1] = (double)((long double)S / (LD * LD) - gap);
        f.fval[i - 1] = (double)((long double)S / (LD * LD));
    }
}

void fw_run(Graph& g, int mode, int iters, bool want_gap, hipStream_t s) {
    fw_prepare(g, mode, iters, s);
    SweepPlan& p = plan_of(g, mode);
    FwState& f = g.fw[mode_slot(mode)];
    const int B = g.idbits;
    const int64_t n = g.n;
    const bool one = iters > 0 && fw_fits_one(g, mode);  // one launch for all iterations
    if (n > 0 && !one) {
        const int32_t* cnt = (mode == 2) ? g.deg.p : (mode == 3 ? g.tcount.p : g.qcount.p);
        k_init_keys<<<grid_for(n, 256), 256, 0, s>>>(cnt, mode == 3 ? 2 : 1, g.orig_of.p, n, B, f.K[0].p, f.K[1].p,
                                                    codes_of(g, mode, 0),
                                                    f.Q[0].p, f.Q[1].p);
        LDS_HIP(hipGetLastError());
    }
    f.cur = 0;
    g.sg[mode_slot(mode)].valid = false;
    const unsigned blocks = sweep_blocks(p);
    const unsigned gblocks = blocks + finish_grid(p) + push_grid(p);  // gap partial sums per iteration
    const size_t npart = want_gap ? (size_t)iters * (one ? 1 : gblocks) * 4 : 0;
    if (f.partial.n < npart) f.partial.alloc(npart, s);
    SweepArgs a;
    fill_sweep_args(g, p, a);
    if (p.n_push > 0 && !one) use_push(p, f, blocks, a, s);
    if (!f.ev[0]) {
        LDS_HIP(hipEventCreate(&f.ev[0]));
        LDS_HIP(hipEventCreate(&f.ev[1]));
    }
    LDS_HIP(hipEventRecord(f.ev[0], s));
    f.launches = 0;
    if (one) {
        fw_run_one(g, mode, iters, want_gap ? f.partial.p : nullptr, s);
        f.cur = iters & 1;
        f.launches = iters;
    }
    for (int i = 1; i <= iters && blocks > 0 && p.nrows > 0 && !one; ++i) {
        sweep_iteration(g, f, p, a, mode, i, blocks, want_gap ? f.partial.p + (size_t)(i - 1) * gblocks * 4 : nullptr,
                        s);
        ++f.launches;
    }
    LDS_HIP(hipEventRecord(f.ev[1], s));
    f.iters = iters;
    f.ran = true;
    f.timed = true;
    f.gap.clear();
    f.lb.clear();
    f.fval.clear();
    if (want_gap && iters > 0) {
        std::vector<uint64_t> sums((size_t)iters * 4, 0);
        if (one) {
            LDS_HIP(hipMemcpyAsync(sums.data(), f.partial.p, sums.size() * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
            LDS_HIP(hipStreamSynchronize(s));
        } else if (blocks > 0 && p.nrows > 0) {
            DBuf<uint64_t> out;
            out.alloc((size_t)iters * 4, s);
            k_gap_reduce<<<iters, 256, 0, s>>>(f.partial.p, gblocks, out.p);
            LDS_HIP(hipGetLastError());
            LDS_HIP(hipMemcpyAsync(sums.data(), out.p, out.bytes(), hipMemcpyDeviceToHost, s));
            LDS_HIP(hipStreamSynchronize(s));
        }
        fw_gap_from_sums(f, mode, iters, sums.data());
    }
}

namespace {

// gap of iteration j + 1 at r^(j) from the exact sums (sum A^2, sum of the
// patterns' minimum A), over D_j = c (j+1)(j+2):
// gap = 2 (sum A^2 - D_j sum min A) / D_j^2, rounded to FP64 on the device
__global__ void k_gap_values(const uint64_t* sums, int iters, uint64_t c, double* gap) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= iters) return;
    const u128 S = ((u128)sums[4 * j + 1] << 64) | sums[4 * j];
    const u128 M = ((u128)sums[4 * j + 3] << 64) | sums[4 * j + 2];
    const uint64_t D = c * (uint64_t)(j + 1) * (uint64_t)(j + 2);
    const u128 num = S - (u128)D * M;
    const double nd = (double)(uint64_t)(num >> 64) * 18446744073709551616.0 + (double)(uint64_t)num;
    const double Dd = (double)D;
    gap[j] = 2.0 * nd / (Dd * Dd);
}

// this device's copy of the scratch array, looked up once per device with
// that device current
uint64_t* scratch_on_current_device() {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static uint64_t* ptr[kMaxDev] = {};
    int dev = 0;
    LDS_HIP(hipGetDevice(&dev));
    LDS_CHECK(dev >= 0 && dev < kMaxDev, ST_DEVICE, "device index out of range for the scratch table");
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        LDS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        LDS_CHECK(p != nullptr, ST_DEVICE, "hipGetSymbolAddress returned no address for the scratch array");
        ptr[dev] = (uint64_t*)p;
    }
    return ptr[dev];
}

}  // namespace


void fw_run_noalloc(Graph& g, int mode, int iters, float* r32_dev, double* gap_host, hipStream_t s) {
    LDS_CHECK(mode >= 2 && mode <= 4, ST_INVALID, "mode must be LDS_EDGE, LDS_TRIANGLE or LDS_CLIQUE4");
    LDS_CHECK(iters >= 0, ST_INVALID, "iters must be >= 0");
    LDS_CHECK(mode != 3 || g.T >= 0, ST_INVALID, "triangles are not listed: run lds_frank_wolfe (or lds_triangles) first");
    LDS_CHECK(mode != 4 || g.Q4 >= 0, ST_INVALID, "4-cliques are not listed: run lds_frank_wolfe (or lds_cliques4) first");
    const SweepPlan& p = plan_of(g, mode);
    FwState& f = g.fw[mode_slot(mode)];
    const int B = g.idbits;
    const u128 amax = fw_max_numerator(g, mode, iters);
    LDS_CHECK(B < 64 && (amax >> (64 - B)) == 0, ST_OVERFLOW, "exact load numerator would overflow the 64-bit key");
    const int64_t n = g.n;
    LDS_CHECK(f.K[0].n == (size_t)n && f.K[1].n == (size_t)n && f.Q[0].n == (size_t)n && f.Q[1].n == (size_t)n &&
                  f.bits.n >= (size_t)iters * (size_t)p.total_words,
              ST_INVALID,
              "Frank-Wolfe state is not sized for this many iterations: run lds_frank_wolfe with at least iters "
              "iterations on this graph and mode first");
    const unsigned blocks = sweep_grid();
    const unsigned gblocks = blocks + finish_grid(p);
    const bool gap = gap_host != nullptr && iters > 0;
    const size_t words = gap ? (size_t)iters * ((size_t)gblocks * 4 + 5) : 0;
    LDS_CHECK(words <= kScratchWords, ST_INVALID,
              "iters exceeds the no-allocation limit with the gap (" +
                  std::to_string(kScratchWords / ((size_t)gblocks * 4 + 5)) + " iterations for this graph)");
    uint64_t* sc = scratch_on_current_device();
    uint64_t* partial = sc;
    uint64_t* sums = sc + (size_t)iters * gblocks * 4;
    double* gapv = reinterpret_cast<double*>(sums + (size_t)iters * 4);
    if (n > 0) {
        const int32_t* cnt = (mode == 2) ? g.deg.p : (mode == 3 ? g.tcount.p : g.qcount.p);
        k_init_keys<<<grid_for(n, 256), 256, 0, s>>>(cnt, mode == 3 ? 2 : 1, g.orig_of.p, n, B, f.K[0].p, f.K[1].p,
                                                    codes_of(g, mode, 0),
                                                    f.Q[0].p, f.Q[1].p);
        LDS_HIP(hipGetLastError());
    }
    f.cur = 0;
    g.sg[mode_slot(mode)].valid = false;
    SweepArgs a;
    fill_sweep_args(g, p, a);
    const bool any = blocks > 0 && p.nrows > 0;
    for (int i = 1; i <= iters && any; ++i)
        sweep_iteration(g, f, p, a, mode, i, blocks, gap ? partial + (size_t)(i - 1) * gblocks * 4 : nullptr, s);
    f.iters = iters;
    f.ran = true;
    f.timed = false;
    f.launches = any ? iters : 0;
    f.gap.clear();
    f.lb.clear();
    f.fval.clear();
    if (n > 0 && r32_dev) {
        k_loads<<<grid_for(n, 256), 256, 0, s>>>(f.K[f.cur].p, g.orig_of.p, n, B, (double)denom(mode, iters), r32_dev,
                                                 nullptr);
        LDS_HIP(hipGetLastError());
    }
    if (gap) {
        if (any) {
            k_gap_reduce<<<iters, 256, 0, s>>>(partial, gblocks, sums);
            LDS_HIP(hipGetLastError());
            k_gap_values<<<grid_for(iters, 256), 256, 0, s>>>(sums, iters, denom(mode, 0) / 2, gapv);
            LDS_HIP(hipGetLastError());
            LDS_HIP(hipMemcpyAsync(gap_host, gapv, (size_t)iters * sizeof(double), hipMemcpyDeviceToHost, s));
            LDS_HIP(hipStreamSynchronize(s));
        } else {
            for (int i = 0; i < iters; ++i) gap_host[i] = 0.0;
        }
    }
}

void fw_loads(const Graph& g, int mode, float* r32_dev, double* r64_host, uint64_t* A_host, hipStream_t s) {
    const FwState& f = g.fw[mode_slot(mode)];
    const int64_t n = g.n;
    if (n == 0) return;
    LDS_CHECK(f.ran && f.K[0].n == (size_t)n, ST_INVALID, "no Frank-Wolfe state: call lds_frank_wolfe first");
    const double D = (double)denom(mode, f.iters);
    DBuf<uint64_t> A;
    if (r64_host || A_host) A.alloc(n, s);
    k_loads<<<grid_for(n, 256), 256, 0, s>>>(f.K[f.cur].p, g.orig_of.p, n, g.idbits, D, r32_dev, A.p);
    LDS_HIP(hipGetLastError());
    if (A.p) {
        std::vector<uint64_t> h(n);
        LDS_HIP(hipMemcpyAsync(h.data(), A.p, n * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
        LDS_HIP(hipStreamSynchronize(s));
        for (int64_t i = 0; i < n; ++i) {
            if (A_host) A_host[i] = h[i];
            if (r64_host) r64_host[i] = (double)h[i] / D;
        }
    }
}

void fw_splits(const Graph& g, int mode, int32_t* verts_host, uint64_t* num_host, hipStream_t s) {
    const FwState& f = g.fw[mode_slot(mode)];
    const SweepPlan& p = plan_of(g, mode);
    const int64_t ns = p.nslots;
    if (ns == 0) return;
    LDS_CHECK(f.ran && f.K[0].n == (size_t)g.n, ST_INVALID, "no Frank-Wolfe state: call lds_frank_wolfe first");
    const int H = mode;
    DBuf<int32_t> v;
    DBuf<uint64_t> a;
    v.alloc((size_t)ns * H, s);
    a.alloc(ns, s);
    // a0 = D_0 / h; inc_i = D_i - D_{i-1} = incm (i+1) with incm = inc_1 / 2
    const uint64_t a0 = denom(mode, 0) / (uint64_t)H, incm = (denom(mode, 1) - denom(mode, 0)) / 2;
    if (mode == 2) {
        k_splits<2, false><<<grid_for(ns, 256), 256, 0, s>>>(p.rp, p.rid, p.py, p.bitbase.p, p.nrows, ns, f.bits.p,
                                                      p.total_words, f.iters, a0, incm, g.orig_of.p, v.p, a.p);
        const HeavyPlan& h = p.heavy;
        if (h.positions > 0)
            k_splits_heavy<<<grid_for(h.positions, 256), 256, 0, s>>>(h.csr.p, h.pay.p, h.positions, h.word0, p.rp,
                                                                      p.nrows, p.py, f.bits.p, p.total_words,
                                                                      f.iters, a0, incm, g.orig_of.p, v.p, a.p);
        if (p.n_push > 0)  // the hub rows' slots against non-hub vertices, from their mirror slots
            k_push_mirror<uint64_t><<<(unsigned)std::min<int64_t>(p.n_push, 4096), 256, 0, s>>>(
                p.rp, p.py, p.hub_pre.p, p.n_push, denom(mode, f.iters), a.p);
    }
    else if (mode == 3)
        k_splits<3, false><<<grid_for(ns, 256), 256, 0, s>>>(p.rp, p.rid, p.py, p.bitbase.p, p.nrows, ns, f.bits.p,
                                                      p.total_words, f.iters, a0, incm, g.orig_of.p, v.p, a.p);
    else
        (p.packed ? k_splits<4, true> : k_splits<4, false>)<<<grid_for(ns, 256), 256, 0, s>>>(
            p.rp, p.rid, p.py, p.bitbase.p, p.nrows, ns, f.bits.p, p.total_words, f.iters, a0, incm, g.orig_of.p, v.p,
            a.p);
    LDS_HIP(hipGetLastError());
    LDS_HIP(hipMemcpyAsync(verts_host, v.p, v.bytes(), hipMemcpyDeviceToHost, s));
    LDS_HIP(hipMemcpyAsync(num_host, a.p, a.bytes(), hipMemcpyDeviceToHost, s));
    LDS_HIP(hipStreamSynchronize(s));
}

}  // namespace lds
