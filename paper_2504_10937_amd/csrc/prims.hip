// Device primitives for gfx950: exclusive prefix sums and a stable LSD radix
// sort (8-bit digits, 4096-key tiles, wave64 ballot matching for the stable
// in-tile ranks).  Used by graph ingest, the triangle incidence build and the
// sort of converged loads (the first step of Alg. 2).
#include "common.hpp"
#include "wave.hpp"

namespace lds {

namespace {

constexpr int kThreads = 256;
constexpr int kItems = 16;
constexpr int kTile = kThreads * kItems;  // 4096
constexpr int64_t kSerialTiles = 3;  // tiles that one workgroup scans in the time of the three launches for more

// inclusive scan over the 256 threads of a block; `total` gets the block sum
__device__ inline uint64_t block_incl_scan(uint64_t x, uint64_t* sh, uint64_t& total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    x = (uint64_t)wave::scan((int64_t)x, (int64_t)0, [](int64_t u, int64_t v) { return u + v; });
    if (lane == 63) sh[w] = x;
    __syncthreads();
    uint64_t pre = 0;
    for (int i = 0; i < w; ++i) pre += sh[i];
    total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return x + pre;
}

template <class T>
__global__ __launch_bounds__(kThreads) void k_tile_sums(const T* in, int64_t n, uint64_t* sums) {
    __shared__ uint64_t sh[4];
    const int64_t base = (int64_t)blockIdx.x * kTile;
    uint64_t acc = 0;
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        int64_t i = base + (int64_t)k * kThreads + threadIdx.x;
        if (i < n) acc += (uint64_t)in[i];
    }
    uint64_t tot;
    block_incl_scan(acc, sh, tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Exclusive scan of `tiles` consecutive tiles per workgroup (one when their
// offsets are given).  A tile is loaded with all its reads in flight, turned
// in LDS so that a thread holds kItems consecutive entries (padded: threads
// start one bank apart), scanned with one block scan, and turned back for the
// stores.  Bound: latency on one tile, bandwidth on many.  A block scan (and
// two barriers) per 256 entries took 10 us for one tile; now 3.0 us.
template <class T>
__global__ __launch_bounds__(kThreads) void k_tile_scan(const T* in, uint64_t* out, int64_t n,
                                                        const uint64_t* tile_off, uint64_t* total_dev,
                                                        int64_t ntiles, int tiles) {
    __shared__ uint64_t sh[4];
    __shared__ uint64_t buf[kTile + kThreads];
    uint64_t carry = tile_off ? tile_off[blockIdx.x] : 0;
    for (int t = 0; t < tiles; ++t) {
        const int64_t tile = (int64_t)blockIdx.x * tiles + t, base = tile * kTile;
        if (tile >= ntiles) break;
        uint64_t x[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = base + (int64_t)k * kThreads + threadIdx.x;
            x[k] = (i < n) ? (uint64_t)in[i] : 0;
        }
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int e = k * kThreads + threadIdx.x;
            buf[e + e / kItems] = x[k];
        }
        __syncthreads();
        uint64_t* mine = buf + threadIdx.x * (kItems + 1);
        uint64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            x[k] = mine[k];
            sum += x[k];
        }
        uint64_t tot;
        uint64_t run = carry + block_incl_scan(sum, sh, tot) - sum;
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            mine[k] = run;
            run += x[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int e = k * kThreads + threadIdx.x;
            if (base + e < n) out[base + e] = buf[e + e / kItems];
        }
        carry += tot;
        if (total_dev && tile == ntiles - 1 && threadIdx.x == 0) *total_dev = carry;
        if (t + 1 < tiles) __syncthreads();  // buf is rewritten by the next tile
    }
}

template <class T>
void scan_impl(const T* in, uint64_t* out, int64_t n, uint64_t* total_dev, hipStream_t s) {
    if (n <= 0) {
        if (total_dev) LDS_HIP(hipMemsetAsync(total_dev, 0, sizeof(uint64_t), s));
        return;
    }
    int64_t ntiles = (n + kTile - 1) / kTile;
    if (ntiles <= kSerialTiles) {
        k_tile_scan<T><<<1, kThreads, 0, s>>>(in, out, n, nullptr, total_dev, ntiles, (int)ntiles);
        LDS_HIP(hipGetLastError());
        return;
    }
    DBuf<uint64_t> sums;
    sums.alloc(ntiles, s);
    k_tile_sums<T><<<grid_for(ntiles, 1), kThreads, 0, s>>>(in, n, sums.p);
    LDS_HIP(hipGetLastError());
    scan_impl<uint64_t>(sums.p, sums.p, ntiles, nullptr, s);
    k_tile_scan<T><<<grid_for(ntiles, 1), kThreads, 0, s>>>(in, out, n, sums.p, total_dev, ntiles, 1);
    LDS_HIP(hipGetLastError());
}

// ------------------------------------------------------------- radix sort
// Keys of a pass: an array, or both orientations of every endpoint pair made
// on the fly (key i: pair i / 2, as (a, b) or (b, a)); pairs that are no edge
// (loops, ids out of range) give no key.
struct ArrayKeys {
    const uint64_t* k;
    const uint64_t* n_dev;  // number of keys when the host does not know it, else nullptr
    int64_t n;
    __device__ int64_t count() const { return n_dev ? (int64_t)*n_dev : n; }
    typedef uint64_t Raw;
    __device__ Raw fetch(int64_t i, int64_t nk) const { return i < nk ? k[i] : 0; }
    __device__ bool make(Raw r, int64_t i, int64_t nk, uint64_t& key) const {
        key = r;
        return i < nk;
    }
};
struct PairKeys {
    const int32_t* src;
    const int32_t* dst;
    int64_t np, n;
    int vb, low;  // bits of an id; low bits of a row that lead its key
    unsigned strict;
    unsigned* err;  // bit 0: an id out of range, bit 1: a loop (strict only)
    __device__ int64_t count() const { return 2 * np; }
    typedef int2 Raw;
    __device__ Raw fetch(int64_t i, int64_t nk) const {
        return i < nk ? make_int2(src[i >> 1], dst[i >> 1]) : make_int2(0, 0);
    }
    __device__ bool make(Raw r, int64_t i, int64_t nk, uint64_t& key) const {
        key = 0;
        if (i >= nk) return false;
        const int64_t a = r.x, b = r.y;
        if (a < 0 || b < 0 || a >= n || b >= n || a == b) {
            const unsigned e = a != b || a < 0 || a >= n ? 1u : 2u * strict;
            if (e) atomicOr(err, e);
            return false;
        }
        const uint64_t row = (uint64_t)((i & 1) ? b : a), nb = (uint64_t)((i & 1) ? a : b);
        const uint64_t lead = ((row & ((1ull << low) - 1)) << (vb - low)) | (row >> low);
        key = (lead << vb) | nb;
        return true;
    }
};

// NW waves per workgroup, a tile of NW * 1024 keys.  Long sorts take 8 waves
// and put the tile into digit order in LDS before the stores, so that a digit's
// keys (256 bytes in the mean) leave as whole lines; with a 4-wave tile the same
// reordering gives nothing (its runs of 128 bytes straddle lines that another
// workgroup completes).  Ingest of 2.1e8 keys with two passes: 13.4 ms by
// unordered 16-wave tiles, 12.6 by ordered ones, 12.2 by ordered 8-wave tiles.
// Shorter sorts take 4 waves, to give every compute unit a tile.
constexpr int64_t kWideFrom = (int64_t)1 << 23;

template <int NW, class KEYS>
__global__ __launch_bounds__(NW * 64) void k_radix_hist(KEYS keys, int shift, uint64_t* hist, int64_t nblocks) {
    constexpr int NT = NW * 64;
    __shared__ uint32_t cnt[256];
    if (threadIdx.x < 256) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (NT * kItems), nk = keys.count();
    typename KEYS::Raw raw[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) raw[k] = keys.fetch(base + (int64_t)k * NT + threadIdx.x, nk);
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        uint64_t key;
        if (keys.make(raw[k], base + (int64_t)k * NT + threadIdx.x, nk, key))
            atomicAdd(&cnt[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256) hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = cnt[threadIdx.x];
}

template <int NW, class KEYS, bool VALS>
__global__ __launch_bounds__(NW * 64) void k_radix_scatter(KEYS keys, const uint32_t* vin, uint64_t* kout,
                                                           uint32_t* vout, int shift, const uint64_t* offs,
                                                           int64_t nblocks) {
    constexpr int NT = NW * 64;
    __shared__ uint32_t wcnt[NW][256];
    __shared__ uint64_t gofs[256];
    __shared__ uint32_t lofs[257];
    extern __shared__ uint64_t stage[];  // NW > 4: the tile in digit order
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < NW * 256; i += NT) (&wcnt[0][0])[i] = 0;
    if (threadIdx.x < 256) gofs[threadIdx.x] = offs[(int64_t)threadIdx.x * nblocks + blockIdx.x];
    __syncthreads();
    // wave w owns the contiguous range [base, base + 1024) of the tile and
    // walks it in 16 rounds of 64 consecutive keys: rank order = key order
    const int64_t base = (int64_t)blockIdx.x * (NT * kItems) + (int64_t)w * (kItems * 64), nk = keys.count();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t key[kItems];
    uint32_t val[kItems];
    uint32_t rank[kItems];
    uint32_t in = 0;  // bit k: key k is one
    {
        typename KEYS::Raw raw[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int64_t i = base + (int64_t)k * 64 + lane;
            raw[k] = keys.fetch(i, nk);
            if (VALS) val[k] = i < nk ? vin[i] : 0;
        }
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            if (keys.make(raw[k], base + (int64_t)k * 64 + lane, nk, key[k])) in |= 1u << k;
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const bool valid = (in >> k) & 1u;
        const uint32_t d = (uint32_t)(key[k] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            uint64_t bb = __ballot((d >> b) & 1u);
            peers &= ((d >> b) & 1u) ? bb : ~bb;
        }
        const uint32_t r = (uint32_t)__popcll(peers & lt);
        uint32_t c = 0;
        if (valid) c = wcnt[w][d];
        rank[k] = c + r;
        if (valid && r == 0) wcnt[w][d] = c + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    {
        const int d = threadIdx.x;
        uint32_t run = 0;
        if (threadIdx.x < 256) {
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                uint32_t t = wcnt[q][d];
                wcnt[q][d] = run;
                run += t;
            }
        }
        if (NW > 4) {  // first place of each digit in the tile
            __shared__ uint32_t wsum[4];
            uint32_t inc = 0;
            if (threadIdx.x < 256) {
                inc = (uint32_t)wave::scan((int64_t)run, (int64_t)0, [](int64_t u, int64_t v) { return u + v; });
                if (lane == 63) wsum[w] = inc;
            }
            __syncthreads();
            if (threadIdx.x < 256) {
                uint32_t pre = 0;
                for (int q = 0; q < w; ++q) pre += wsum[q];
                lofs[d] = pre + inc - run;
                if (d == 255) lofs[256] = pre + inc;
            }
        }
    }
    __syncthreads();
    if constexpr (NW > 4) {
#pragma unroll
        for (int k = 0; k < kItems; ++k)
            if ((in >> k) & 1u) {
                const uint32_t d = (uint32_t)(key[k] >> shift) & 255u;
                rank[k] += lofs[d] + wcnt[w][d];
                stage[rank[k]] = key[k];
            }
        __syncthreads();
        const int total = (int)lofs[256];
        uint64_t pos[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int i = k * NT + (int)threadIdx.x;
            if (i < total) {
                const uint64_t x = stage[i];
                const uint32_t d = (uint32_t)(x >> shift) & 255u;
                pos[k] = gofs[d] + (uint32_t)i - lofs[d];
                kout[pos[k]] = x;
            }
        }
        if (VALS) {
            __syncthreads();
            uint32_t* sv = reinterpret_cast<uint32_t*>(stage);
#pragma unroll
            for (int k = 0; k < kItems; ++k)
                if ((in >> k) & 1u) sv[rank[k]] = val[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kItems; ++k) {
                const int i = k * NT + (int)threadIdx.x;
                if (i < total) vout[pos[k]] = sv[i];
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        if ((in >> k) & 1u) {
            const uint32_t d = (uint32_t)(key[k] >> shift) & 255u;
            const uint64_t pos = gofs[d] + wcnt[w][d] + rank[k];
            kout[pos] = key[k];
            if (VALS) vout[pos] = val[k];
        }
    }
}

constexpr int kWideWaves = 8;
int64_t radix_blocks(int64_t n) {
    const int64_t tile = (n >= kWideFrom ? kWideWaves : 4) * 1024;
    return (n + tile - 1) / tile;
}

template <int NW, class KEYS, bool VALS>
void launch_scatter(const KEYS& keys, const uint32_t* vin, uint64_t* kout, uint32_t* vout, int shift,
                    const uint64_t* hist, int64_t nblocks, hipStream_t s) {
    const size_t lds = NW > 4 ? (size_t)NW * 1024 * sizeof(uint64_t) : 0;
    if (lds)
        LDS_HIP(hipFuncSetAttribute((const void*)k_radix_scatter<NW, KEYS, VALS>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    k_radix_scatter<NW, KEYS, VALS><<<grid_for(nblocks, 1), NW * 64, lds, s>>>(keys, vin, kout, vout, shift, hist,
                                                                              nblocks);
    LDS_HIP(hipGetLastError());
}

template <int NW, class KEYS>
void radix_pass_waves(const KEYS& keys, const uint32_t* vin, uint64_t* kout, uint32_t* vout, int64_t n, int shift,
                      uint64_t* hist, uint64_t* total, hipStream_t s) {
    const int64_t nblocks = radix_blocks(n);
    k_radix_hist<NW><<<grid_for(nblocks, 1), NW * 64, 0, s>>>(keys, shift, hist, nblocks);
    LDS_HIP(hipGetLastError());
    exclusive_scan_u64(hist, hist, 256 * nblocks, total, s);
    if (vin)
        launch_scatter<NW, KEYS, true>(keys, vin, kout, vout, shift, hist, nblocks, s);
    else
        launch_scatter<NW, KEYS, false>(keys, nullptr, kout, nullptr, shift, hist, nblocks, s);
}

// one pass over up to n keys (more precisely keys.count(), on the device);
// hist: 256 * radix_blocks(n) words; total: the number of keys, optional
template <class KEYS>
void radix_pass(const KEYS& keys, const uint32_t* vin, uint64_t* kout, uint32_t* vout, int64_t n, int shift,
                uint64_t* hist, uint64_t* total, hipStream_t s) {
    if (n >= kWideFrom)
        radix_pass_waves<kWideWaves>(keys, vin, kout, vout, n, shift, hist, total, s);
    else
        radix_pass_waves<4>(keys, vin, kout, vout, n, shift, hist, total, s);
}

// The whole sort of at most kTile keys by one workgroup: the passes of
// k_radix_scatter with the keys (and payloads) in LDS, so that a small sort
// is one launch (5 us for 544 keys, 2 passes) instead of three per pass (17 us).
template <bool VALS>
__global__ __launch_bounds__(kThreads) void k_radix_small(uint64_t* keys, uint32_t* vals, int n, int begin_bit,
                                                          int end_bit) {
    __shared__ uint64_t lk[kTile];
    __shared__ uint32_t lv[VALS ? kTile : 1];
    __shared__ uint32_t wcnt[4][256];
    __shared__ uint32_t wsum[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // wave w owns the run of `rounds` * 64 consecutive keys from w * rounds * 64
    const int rounds = (n + kThreads - 1) / kThreads;
    uint64_t key[kItems];
    uint32_t val[kItems];
    uint32_t rank[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = (w * rounds + k) * 64 + lane;
        const bool valid = k < rounds && i < n;
        key[k] = valid ? keys[i] : 0;
        val[k] = (VALS && valid) ? vals[i] : 0;
    }
    for (int shift = begin_bit; shift < end_bit; shift += 8) {
        for (int i = threadIdx.x; i < 4 * 256; i += kThreads) (&wcnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const bool valid = k < rounds && (w * rounds + k) * 64 + lane < n;
            if (__ballot(valid) == 0) continue;
            const uint32_t d = (uint32_t)(key[k] >> shift) & 255u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t bb = __ballot((d >> b) & 1u);
                peers &= ((d >> b) & 1u) ? bb : ~bb;
            }
            const uint32_t r = (uint32_t)__popcll(peers & lt);
            uint32_t c = 0;
            if (valid) c = wcnt[w][d];
            rank[k] = c + r;
            if (valid && r == 0) wcnt[w][d] = c + (uint32_t)__popcll(peers);
        }
        __syncthreads();
        {  // digit d's first place, then each wave's within it
            const int d = threadIdx.x;
            uint32_t c[4], tot = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = tot;
                tot += wcnt[q][d];
            }
            const uint32_t inc =
                (uint32_t)wave::scan((int64_t)tot, (int64_t)0, [](int64_t u, int64_t v) { return u + v; });
            if (lane == 63) wsum[w] = inc;
            __syncthreads();
            uint32_t first = inc - tot;
            for (int q = 0; q < w; ++q) first += wsum[q];
#pragma unroll
            for (int q = 0; q < 4; ++q) wcnt[q][d] = first + c[q];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            if (k < rounds && (w * rounds + k) * 64 + lane < n) {
                const uint32_t pos = wcnt[w][(uint32_t)(key[k] >> shift) & 255u] + rank[k];
                lk[pos] = key[k];
                if (VALS) lv[pos] = val[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
            const int i = (w * rounds + k) * 64 + lane;
            if (k < rounds && i < n) {
                key[k] = lk[i];
                if (VALS) val[k] = lv[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int i = (w * rounds + k) * 64 + lane;
        if (k < rounds && i < n) {
            keys[i] = key[k];
            if (VALS) vals[i] = val[k];
        }
    }
}

}  // namespace

void exclusive_scan_u64(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* total_dev, hipStream_t s) {
    scan_impl<uint64_t>(in, out, n, total_dev, s);
}
void exclusive_scan_u32_to_u64(const uint32_t* in, uint64_t* out, int64_t n, uint64_t* total_dev,
                               hipStream_t s) {
    scan_impl<uint32_t>(in, out, n, total_dev, s);
}

void radix_sort_u64(DBuf<uint64_t>& keys, DBuf<uint32_t>* vals, int64_t n, int begin_bit, int end_bit,
                    DBuf<uint64_t>& tmp_keys, DBuf<uint32_t>* tmp_vals, hipStream_t s) {
    if (n <= 1 || end_bit <= begin_bit) return;
    if (n <= kTile) {
        if (vals)
            k_radix_small<true><<<1, kThreads, 0, s>>>(keys.p, vals->p, (int)n, begin_bit, end_bit);
        else
            k_radix_small<false><<<1, kThreads, 0, s>>>(keys.p, nullptr, (int)n, begin_bit, end_bit);
        LDS_HIP(hipGetLastError());
        return;
    }
    DBuf<uint64_t> hist;
    hist.alloc((size_t)256 * radix_blocks(n), s);
    for (int shift = begin_bit; shift < end_bit; shift += 8) {
        radix_pass(ArrayKeys{keys.p, nullptr, n}, vals ? vals->p : nullptr, tmp_keys.p, vals ? tmp_vals->p : nullptr, n,
                   shift, hist.p, nullptr, s);
        std::swap(keys, tmp_keys);
        if (vals) std::swap(*vals, *tmp_vals);
    }
    // hist is released at scope exit: either to the stream-ordered caching
    // allocator of the caller, or through hipFree, which synchronises.
}

const uint64_t* bucket_pairs(const int32_t* src, const int32_t* dst, int64_t np, int64_t n, int vb, int bits,
                             bool strict, uint64_t* ka, uint64_t* kb, uint64_t* count_dev, unsigned* err,
                             hipStream_t s) {
    DBuf<uint64_t> hist;
    hist.alloc((size_t)256 * radix_blocks(2 * np), s);
    const int shift = 2 * vb - bits;
    radix_pass(PairKeys{src, dst, np, n, vb, bits, strict ? 1u : 0u, err}, nullptr, ka, nullptr, 2 * np, shift, hist.p, count_dev, s);
    if (bits <= 8) return ka;
    radix_pass(ArrayKeys{ka, count_dev, 0}, nullptr, kb, nullptr, 2 * np, shift + 8, hist.p, nullptr, s);
    return kb;
}

}  // namespace lds
