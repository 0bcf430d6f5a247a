// Batched Frank-Wolfe (Alg. 1 / Alg. 6) over many independent graphs in one
// persistent kernel launch, captured once into a hipGraph and replayed.
//
// Each workgroup takes whole graphs from a device work queue (an atomic
// counter over the items, which are ordered longest-first) and runs all the
// iterations of a graph by itself: the iteration barrier is a workgroup
// barrier instead of a kernel boundary, and the keys of a graph with at most
// `kmax` vertices live in LDS for the whole run (two ping-pong buffers), so
// every gather of a neighbour's key is an LDS read.  Larger graphs keep their
// keys in their own device buffers (L2-resident for the sizes admitted here).
//
// The arithmetic, the slot layout and the decision-word layout are those of
// the per-graph sweep: a vertex wins a slot iff its packed key
// (A << B) | (2^B - 1 - orig_id) is below the keys of the pattern's other
// vertices; wins of a row are counted from the decision words; A += inc_i * b.
// So a batched run leaves every graph in exactly the state a per-graph run of
// the same iteration count leaves (keys, decision words, gap sums), and every
// later call (loads, splits, stable groups, top-k) reads it unchanged.
#include <algorithm>
#include <chrono>
#include <cstring>
#include <numeric>

#include "batch.hpp"
#include "wave.hpp"

namespace lds {

namespace {

typedef unsigned __int128 u128;

struct BItem {
    const int32_t* rid;  // compact row -> vertex (nullptr: identity)
    const int64_t* rp;
    const int32_t* py;
    const uint64_t* wdesc;  // per decision word: its slots and first row (word_desc)
    const uint64_t* head;
    const int64_t* bitbase;
    const int32_t* cnt;     // deg (edges) or triangle count per vertex
    const int32_t* orig_of;
    uint64_t* K0;           // the graph's key buffers
    uint64_t* K1;
    uint64_t* bits;         // iters * total_words decision words
    uint64_t* sums;         // iters * 4 exact gap sums, or nullptr
    float* r_out;           // n loads by caller id, or nullptr
    int32_t chunk_words, total_words, nrows, n_hub;
    int32_t n, h, mult, B, iters, lds_keys;
};

__device__ inline uint64_t readlane64(uint64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

__device__ inline uint64_t fw_inc(int h, int i) {  // D_i - D_{i-1}
    return (uint64_t)(h == 3 ? 6 : 2) * (uint64_t)(i + 1);
}

// 64-slot words in flight per wave.  A batch costs its instructions whether its
// words are there or not: the graphs that run alone in k_fw_one have few words
// a wave (446 slots 2.03 us an iteration with 8, 1.54 with 4; 2.6k 2.78 and
// 2.49; 10k 4.65 and 4.46; 16k 6.42 and 6.51), the largest of a batch, which
// bound its time, many.
constexpr int kBatchWords = 8, kOneWords = 4;
constexpr int kRows = 4;   // rows per thread whose bounds stay in registers over the iterations

// LDS of a workgroup: two key buffers of kmax vertices, then the decision
// words of an iteration (wmax of them; plans with more words read them back
// from memory)
struct Lds {
    uint64_t* keys;
    int32_t kmax;
    uint64_t* words;
    int32_t wmax;
    uint64_t (*red)[4];
};

// One graph, all iterations, by one workgroup; the keys ping-pong between Ka
// and Kb (LDS when KLDS, else the graph's own buffers).  An iteration has two
// phases.  Decision words: every wave takes an equal run of them, kG at a time
// with their payload reads in flight together and every key an LDS read; a
// word's slots and first row are scalars (word_desc), whatever rows or chunks
// it belongs to.  Rows: a thread per row (a wave per row of more than kChunk
// slots) counts the row's wins in the words and writes its key.  Bound: LDS
// reads (two or three 8-byte keys per slot) and issue.  One word at a time by
// chunks, with keys through generic pointers and a barrier pair per hub row,
// 768 graphs (half edge, half triangle density, n <= 5000) took 21 ms; now
// 8.0 ms.
template <int H, int NT, bool KLDS, int kG>
__device__ void run_graph(const BItem& it, uint64_t* Ka, uint64_t* Kb, const Lds& l) {
    constexpr int NW = NT / 64;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int B = it.B;
    const uint64_t idm = (1ull << B) - 1ull;
    const uint64_t le = (lane == 63) ? ~0ull : ((2ull << lane) - 1ull);
    const int words = it.total_words;
    const bool wlds = words <= l.wmax;
    // a wave's run of words, in whole batches
    const int per = ((words + NW - 1) / NW + kG - 1) / kG * kG;
    const int wb = min(words, w * per), we = min(words, wb + per);
    // initial keys in both buffers: vertices without slots never change
    for (int u = threadIdx.x; u < it.n; u += NT) {
        const uint64_t k = (((uint64_t)it.cnt[u] * (uint64_t)it.mult) << B) | (idm - (uint64_t)it.orig_of[u]);
        Ka[u] = k;
        Kb[u] = k;
    }
    struct Row {
        int32_t bit, len, u;
    };
    auto load_row = [&](int r) {
        Row x{0, 0, 0};
        if (r < it.nrows) {
            x.bit = (int32_t)it.bitbase[r];
            x.len = (int32_t)(it.rp[r + 1] - it.rp[r]);
            x.u = it.rid ? it.rid[r] : r;
        }
        return x;
    };
    Row mine[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) mine[k] = load_row(it.n_hub + (int)threadIdx.x + k * NT);
    // the run's first 64 word descriptors and row-start flags
    const uint64_t wd0 = wb + lane < we ? it.wdesc[wb + lane] : 0ull;
    const uint64_t hd0 = wb + lane < min(we, it.chunk_words) ? it.head[wb + lane] : 0ull;
    __syncthreads();
    int cur = 0;
    for (int i = 1; i <= it.iters; ++i) {
        const uint64_t* Kin = cur ? Kb : Ka;
        uint64_t* Kout = cur ? Ka : Kb;
        const uint64_t inc = fw_inc(H, i);
        uint64_t* bits = it.bits + (int64_t)(i - 1) * it.total_words;
        // ---- decision words
        for (int b0 = wb; b0 < we; b0 += 64) {
            const int x = b0 + lane;
            uint64_t wd = wd0, hd = hd0;
            if (b0 > wb) {
                wd = x < we ? it.wdesc[x] : 0ull;
                hd = x < min(we, it.chunk_words) ? it.head[x] : 0ull;
            }
            uint64_t mybits = 0;
            const int nb = min(64, we - b0);
            for (int t0 = 0; t0 < nb; t0 += kG) {
                int32_t v[kG][H - 1], uu[kG];
                bool win[kG];
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    // past the run's end: word 0 of nothing (no lane is in)
                    const uint64_t dsc = readlane64(wd, t0 + j), hw = readlane64(hd, t0 + j);
                    const int nin = t0 + j < nb ? word_slots(dsc) : 0;
                    win[j] = lane < nin;
                    uu[j] = word_row(dsc) + (int32_t)__popcll(hw & le);
                    const int32_t* py = it.py + (int64_t)word_slot(dsc) * (H - 1);
                    if (H == 2) {
                        v[j][0] = win[j] ? py[lane] : 0;
                    } else {
                        const int2 y = win[j] ? reinterpret_cast<const int2*>(py)[lane] : make_int2(0, 0);
                        v[j][0] = y.x;
                        v[j][H - 2] = y.y;
                    }
                }
                if (it.rid) {
#pragma unroll
                    for (int j = 0; j < kG; ++j) uu[j] = win[j] ? it.rid[uu[j]] : 0;
                } else {
#pragma unroll
                    for (int j = 0; j < kG; ++j) uu[j] = win[j] ? uu[j] : 0;
                }
                uint64_t k0[kG], kv[kG][H - 1];
#pragma unroll
                for (int j = 0; j < kG; ++j) {
                    k0[j] = Kin[uu[j]];
#pragma unroll
                    for (int q = 0; q < H - 1; ++q) kv[j][q] = Kin[v[j][q]];
                }
#pragma unroll
                for (int j = 0; j < kG; ++j) {
#pragma unroll
                    for (int q = 0; q < H - 1; ++q) win[j] = win[j] && k0[j] < kv[j][q];
                    const uint64_t W = __ballot(win[j]);
                    if (lane == t0 + j) mybits = W;
                }
            }
            if (x < we) {
                bits[x] = mybits;
                if (wlds) l.words[x] = mybits;
            }
        }
        __syncthreads();
        // ---- rows
        u128 sq = 0, mn = 0;
        auto word = [&](int x) { return wlds ? l.words[x] : bits[x]; };
        auto update = [&](int32_t u, uint64_t wins) {
            const uint64_t Ku = Kin[u];
            Kout[u] = Ku + ((wins * inc) << B);
            if (it.sums) {
                const uint64_t A = Ku >> B;
                sq += (u128)A * A;
                mn += (u128)A * wins;
            }
        };
        for (int r = w; r < it.n_hub; r += NW) {  // word-aligned
            const Row y = load_row(r);
            uint32_t c = 0;
            for (int q = lane; q < (y.len + 63) / 64; q += 64) c += (uint32_t)__popcll(word((y.bit >> 6) + q));
#pragma unroll
            for (int m = 32; m > 0; m >>= 1) c += (uint32_t)__shfl_xor((int)c, m, 64);
            if (lane == 0) update(y.u, c);
        }
        auto row = [&](const Row& y) {
            uint32_t c = 0;
            const int last = y.bit + y.len - 1;
            for (int wi = y.bit >> 6; wi <= last >> 6; ++wi) {
                const int lo = max(y.bit - wi * 64, 0), hi = min(last + 1 - wi * 64, 64);
                const uint64_t mk = ((hi >= 64) ? ~0ull : ((1ull << hi) - 1ull)) & (~0ull << lo);
                c += (uint32_t)__popcll(word(wi) & mk);
            }
            update(y.u, c);
        };
#pragma unroll
        for (int k = 0; k < kRows; ++k)
            if (mine[k].len > 0) row(mine[k]);
        for (int r = it.n_hub + (int)threadIdx.x + kRows * NT; r < it.nrows; r += NT) row(load_row(r));
        if (it.sums) {
            sq = wave::sum128_lane63(sq);
            mn = wave::sum128_lane63(mn);
            if (lane == 63) {
                l.red[w][0] = (uint64_t)sq;
                l.red[w][1] = (uint64_t)(sq >> 64);
                l.red[w][2] = (uint64_t)mn;
                l.red[w][3] = (uint64_t)(mn >> 64);
            }
        }
        __syncthreads();  // keys of iteration i written, its words read
        cur ^= 1;
        // the waves' sums are read before the next barrier, rewritten after it
        if (it.sums && threadIdx.x == NT - 1) {
            u128 S = 0, M = 0;
            for (int q = 0; q < NW; ++q) {
                S += ((u128)l.red[q][1] << 64) | l.red[q][0];
                M += ((u128)l.red[q][3] << 64) | l.red[q][2];
            }
            uint64_t* o = it.sums + 4 * (int64_t)(i - 1);
            o[0] = (uint64_t)S;
            o[1] = (uint64_t)(S >> 64);
            o[2] = (uint64_t)M;
            o[3] = (uint64_t)(M >> 64);
        }
    }
    // final keys into the graph's buffer number (iters & 1), loads by caller id
    const uint64_t* Kend = cur ? Kb : Ka;
    uint64_t* Kfin = (it.iters & 1) ? it.K1 : it.K0;
    const double D = (double)((uint64_t)(H == 3 ? 3 : 1) * (uint64_t)(it.iters + 1) * (uint64_t)(it.iters + 2));
    for (int u = threadIdx.x; u < it.n; u += NT) {
        const uint64_t k = Kend[u];
        if (KLDS) Kfin[u] = k;
        if (it.r_out) it.r_out[it.orig_of[u]] = (float)((double)(k >> B) / D);
    }
    __syncthreads();  // LDS keys are reused by the next graph
}

template <int NT>
__device__ inline void run_item(const BItem& it, const Lds& l) {
    if (it.lds_keys) {
        if (it.h == 2)
            run_graph<2, NT, true, kBatchWords>(it, l.keys, l.keys + l.kmax, l);
        else
            run_graph<3, NT, true, kBatchWords>(it, l.keys, l.keys + l.kmax, l);
    } else {
        if (it.h == 2)
            run_graph<2, NT, false, kBatchWords>(it, it.K0, it.K1, l);
        else
            run_graph<3, NT, false, kBatchWords>(it, it.K0, it.K1, l);
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_fw_batch(const BItem* __restrict__ items, int32_t count, int32_t* queue,
                                                int32_t kmax, int32_t wmax) {
    extern __shared__ uint64_t dyn[];  // 2 * kmax keys, wmax words
    __shared__ uint64_t red[NT / 64][4];
    __shared__ int32_t next;
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(queue, 1);
        __syncthreads();
        const int32_t idx = next;
        __syncthreads();  // every thread has read `next`
        if (idx >= count) break;
        const BItem it = items[idx];
        run_item<NT>(it, Lds{dyn, kmax, dyn + 2 * (size_t)kmax, wmax, red});
    }
}

// One small graph by one workgroup (fw_run_one): keys and words in LDS
template <int NT>
__global__ __launch_bounds__(NT) void k_fw_one(BItem it) {
    extern __shared__ uint64_t dyn[];
    __shared__ uint64_t red[NT / 64][4];
    const Lds l{dyn, it.n, dyn + 2 * (size_t)it.n, it.total_words, red};
    if (it.h == 2)
        run_graph<2, NT, true, kOneWords>(it, l.keys, l.keys + l.kmax, l);
    else
        run_graph<3, NT, true, kOneWords>(it, l.keys, l.keys + l.kmax, l);
}

__global__ void k_zero_i32(int32_t* p) { *p = 0; }

template <int NT>
void set_lds_limit(size_t bytes) {
    LDS_HIP(hipFuncSetAttribute((const void*)k_fw_batch<NT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
}

template <int NT>
void launch_batch(unsigned grid, size_t lds, hipStream_t s, const BItem* items, int32_t count, int32_t* queue,
                  int32_t kmax, int32_t wmax) {
    k_fw_batch<NT><<<grid, NT, lds, s>>>(items, count, queue, kmax, wmax);
}

int device_cus() {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        LDS_HIP(hipGetDevice(&dev));
        LDS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        if (cus <= 0) cus = 1;
    }
    return cus;
}

// the kernel's view of a graph whose FW buffers are sized for iters
BItem make_item(Graph& g, int mode, int iters, int lds_vertices) {
    const SweepPlan& p = (mode == 2) ? g.edge_plan : g.tri_plan;
    FwState& f = g.fw[mode == 2 ? 0 : 1];
    BItem x;
    std::memset(&x, 0, sizeof(x));
    x.rid = p.rid;
    x.rp = p.rp;
    x.py = p.py;
    x.wdesc = p.wdesc.p;
    x.head = p.head.p;
    x.bitbase = p.bitbase.p;
    x.cnt = (mode == 2) ? g.deg.p : g.tcount.p;
    x.orig_of = g.orig_of.p;
    x.K0 = f.K[0].p;
    x.K1 = f.K[1].p;
    x.bits = f.bits.p;
    x.chunk_words = (int32_t)p.chunk_words;
    x.total_words = (int32_t)p.total_words;
    x.nrows = (int32_t)p.nrows;
    x.n_hub = (int32_t)p.n_hub;
    x.n = (int32_t)g.n;
    x.h = mode;
    x.mult = (mode == 2) ? 1 : 2;
    x.B = g.idbits;
    x.iters = (p.nrows > 0) ? iters : 0;
    x.lds_keys = (g.n <= lds_vertices) ? 1 : 0;
    return x;
}

}  // namespace

// Whether fw_run gives the graph to one workgroup for all iterations: its
// keys fit LDS and a sweep launch would take longer than the workgroup's pass
// over the slots and rows.  Microseconds an iteration of a call, by one
// workgroup and by sweeps: 1500 vertices with 4.0k slots 3.6 and 6.0, 10.0k 4.9
// and 6.1, 12.0k 5.8 and 6.1, 14.0k 6.7 and 6.0; 6000 vertices with 10.0k slots
// 6.1 and 6.4, 12.0k 7.2 and 6.3; triangles of 300 vertices with 11.8k 6.2 and
// 6.0; a clique of 120 (14.3k) 5.4 and 5.7.
namespace {
constexpr size_t kMaxLds = 160 * 1024 - 2048;  // dynamic LDS of a workgroup, beside the reductions
size_t one_lds(const Graph& g, const SweepPlan& p) {
    return ((size_t)2 * (size_t)g.n + (size_t)p.total_words) * sizeof(uint64_t);
}
}  // namespace

bool fw_fits_one(const Graph& g, int mode) {
    if (mode != 2 && mode != 3) return false;
    const SweepPlan& p = plan_of(g, mode);
    return g.n > 0 && g.n <= kOneVertices && p.nrows > 0 && p.nslots + g.n / 4 <= kOneSlots && p.wdesc.p &&
           one_lds(g, p) <= kMaxLds;
}

void fw_run_one(Graph& g, int mode, int iters, uint64_t* sums, hipStream_t s) {
    BItem x = make_item(g, mode, iters, kOneVertices);
    x.sums = sums;
    const size_t lds = one_lds(g, plan_of(g, mode));
    if (x.total_words <= 4 * kOneWords) {  // a batch of words per wave: fewer waves, cheaper barriers
        LDS_HIP(hipFuncSetAttribute((const void*)k_fw_one<256>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kMaxLds));
        k_fw_one<256><<<1, 256, lds, s>>>(x);
    } else {
        LDS_HIP(hipFuncSetAttribute((const void*)k_fw_one<1024>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kMaxLds));
        k_fw_one<1024><<<1, 1024, lds, s>>>(x);
    }
    LDS_HIP(hipGetLastError());
}

int64_t batch_cost(const Graph& g, int mode, int iters) {
    const SweepPlan& p = (mode == 2) ? g.edge_plan : g.tri_plan;
    return (p.nslots + g.n) * (int64_t)std::max(iters, 1);
}

Batch::~Batch() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (cap) (void)hipStreamDestroy(cap);
    if (ev[0]) (void)hipEventDestroy(ev[0]);
    if (ev[1]) (void)hipEventDestroy(ev[1]);
}

void batch_build(Batch& b, hipStream_t s) {
    const int count = (int)b.gs.size();
    const BatchTune& t = b.tune;
    LDS_CHECK(t.threads == 256 || t.threads == 512 || t.threads == 1024, ST_INVALID, "threads must be 256, 512 or 1024");
    LDS_CHECK(t.wg_per_cu >= 1 && t.wg_per_cu <= 8, ST_INVALID, "wg_per_cu must be in [1, 8]");
    LDS_CHECK(t.lds_vertices >= 0 && t.lds_vertices <= 8192, ST_INVALID, "lds_vertices must be in [0, 8192]");
    // FW buffers of every graph, triangle lists, key-width checks
    for (int i = 0; i < count; ++i) fw_prepare(*b.gs[i], b.modes[i], b.iters[i], s);
    // kernel items vs per-graph runs
    b.kernel_items.clear();
    b.plain_items.clear();
    for (int i = 0; i < count; ++i) {
        // graphs whose plans have no word descriptors (large ones) take their
        // own launches
        if (batch_cost(*b.gs[i], b.modes[i], b.iters[i]) <= t.max_kernel_cost &&
            plan_of(*b.gs[i], b.modes[i]).wdesc_built)
            b.kernel_items.push_back(i);
        else
            b.plain_items.push_back(i);
    }
    if (t.longest_first)
        std::stable_sort(b.kernel_items.begin(), b.kernel_items.end(), [&](int x, int y) {
            return batch_cost(*b.gs[x], b.modes[x], b.iters[x]) > batch_cost(*b.gs[y], b.modes[y], b.iters[y]);
        });
    int32_t kmax = 0;
    int64_t wmax = 0;
    for (int i : b.kernel_items) {
        if (b.gs[i]->n <= t.lds_vertices) kmax = std::max<int32_t>(kmax, (int32_t)b.gs[i]->n);
        wmax = std::max(wmax, plan_of(*b.gs[i], b.modes[i]).total_words);
    }
    b.kmax = kmax;
    // the words of an iteration in what LDS the keys leave to each workgroup of a CU
    const int64_t room = ((int64_t)kMaxLds / t.wg_per_cu - (t.wg_per_cu > 1 ? 2048 : 0)) / 8 - 2 * (int64_t)kmax;
    b.wmax = (int32_t)std::max<int64_t>(0, std::min(wmax, room));
    const size_t nk = b.kernel_items.size();
    b.sums.release();
    if (b.want_gap) {
        int64_t tot = 0;
        for (int i : b.kernel_items) tot += 4 * (int64_t)b.iters[i];
        b.sums.alloc((size_t)std::max<int64_t>(tot, 1), s);
    }
    std::vector<BItem> h(nk);
    int64_t soff = 0;
    b.sum_off.assign(nk, 0);
    for (size_t j = 0; j < nk; ++j) {
        const int i = b.kernel_items[j];
        Graph& g = *b.gs[i];
        const int mode = b.modes[i];
        h[j] = make_item(g, mode, b.iters[i], t.lds_vertices);
        h[j].sums = b.want_gap ? b.sums.p + soff : nullptr;
        b.sum_off[j] = soff;
        if (b.want_gap) soff += 4 * (int64_t)b.iters[i];
        h[j].r_out = b.r_out.empty() ? nullptr : b.r_out[i];
        // a graph without patterns keeps its initial keys; its state still
        // records the requested iteration count
    }
    b.items.alloc(std::max<size_t>(nk, 1) * sizeof(BItem), s);
    if (nk) LDS_HIP(hipMemcpyAsync(b.items.p, h.data(), nk * sizeof(BItem), hipMemcpyHostToDevice, s));
    const BItem* items = reinterpret_cast<const BItem*>(b.items.p);
    b.queue.alloc(1, s);
    LDS_HIP(hipStreamSynchronize(s));
    // capture: reset the queue, run the batch kernel
    if (b.exec) {
        (void)hipGraphExecDestroy(b.exec);
        b.exec = nullptr;
    }
    if (b.graph) {
        (void)hipGraphDestroy(b.graph);
        b.graph = nullptr;
    }
    if (b.capture && !b.cap) LDS_HIP(hipStreamCreateWithFlags(&b.cap, hipStreamNonBlocking));
    if (!b.ev[0]) {
        LDS_HIP(hipEventCreate(&b.ev[0]));
        LDS_HIP(hipEventCreate(&b.ev[1]));
    }
    if (nk == 0) return;
    const size_t lds = ((size_t)2 * (size_t)kmax + (size_t)b.wmax) * sizeof(uint64_t);
    const unsigned grid =
        (unsigned)std::min<int64_t>((int64_t)device_cus() * t.wg_per_cu, (int64_t)nk);
    switch (t.threads) {
        case 256: set_lds_limit<256>(lds); break;
        case 512: set_lds_limit<512>(lds); break;
        default: set_lds_limit<1024>(lds); break;
    }
    b.grid = grid;
    b.lds_bytes = lds;
    if (!b.capture) return;
    LDS_HIP(hipStreamBeginCapture(b.cap, hipStreamCaptureModeThreadLocal));
    k_zero_i32<<<1, 1, 0, b.cap>>>(b.queue.p);
    switch (t.threads) {
        case 256: launch_batch<256>(grid, lds, b.cap, items, (int32_t)nk, b.queue.p, kmax, b.wmax); break;
        case 512: launch_batch<512>(grid, lds, b.cap, items, (int32_t)nk, b.queue.p, kmax, b.wmax); break;
        default: launch_batch<1024>(grid, lds, b.cap, items, (int32_t)nk, b.queue.p, kmax, b.wmax); break;
    }
    const hipError_t le = hipGetLastError();
    hipGraph_t gr = nullptr;
    const hipError_t ce = hipStreamEndCapture(b.cap, &gr);
    LDS_HIP(le);
    LDS_HIP(ce);
    b.graph = gr;
    LDS_HIP(hipGraphInstantiate(&b.exec, b.graph, nullptr, nullptr, 0));
}

namespace {
void launch_direct(Batch& b, hipStream_t s) {
    const int32_t nk = (int32_t)b.kernel_items.size();
    if (nk == 0) return;
    const BItem* items = reinterpret_cast<const BItem*>(b.items.p);
    k_zero_i32<<<1, 1, 0, s>>>(b.queue.p);
    switch (b.tune.threads) {
        case 256: launch_batch<256>(b.grid, b.lds_bytes, s, items, nk, b.queue.p, b.kmax, b.wmax); break;
        case 512: launch_batch<512>(b.grid, b.lds_bytes, s, items, nk, b.queue.p, b.kmax, b.wmax); break;
        default: launch_batch<1024>(b.grid, b.lds_bytes, s, items, nk, b.queue.p, b.kmax, b.wmax); break;
    }
    LDS_HIP(hipGetLastError());
}
}  // namespace

void batch_run(Batch& b, hipStream_t s) {
    const int count = (int)b.gs.size();
    // graphs too large for one workgroup: per-graph runs on the same stream
    for (int i : b.plain_items) {
        fw_run(*b.gs[i], b.modes[i], b.iters[i], b.want_gap, s);
        if (!b.r_out.empty() && b.r_out[i]) fw_loads(*b.gs[i], b.modes[i], b.r_out[i], nullptr, nullptr, s);
    }
    LDS_HIP(hipEventRecord(b.ev[0], s));
    if (b.capture) {
        if (b.exec) LDS_HIP(hipGraphLaunch(b.exec, s));
    } else {
        launch_direct(b, s);
    }
    LDS_HIP(hipEventRecord(b.ev[1], s));
    for (size_t j = 0; j < b.kernel_items.size(); ++j) {
        const int i = b.kernel_items[j];
        Graph& g = *b.gs[i];
        const int mode = b.modes[i];
        FwState& f = g.fw[mode == 2 ? 0 : 1];
        f.iters = b.iters[i];
        const SweepPlan& p = (mode == 2) ? g.edge_plan : g.tri_plan;
        f.cur = (p.nrows > 0) ? (b.iters[i] & 1) : 0;
        f.ran = true;
        f.timed = false;
        f.gap.clear();
        f.lb.clear();
        f.fval.clear();
        g.sg[mode == 2 ? 0 : 1].valid = false;
    }
    b.runs++;
    (void)count;
    if (b.want_gap && !b.kernel_items.empty()) {
        std::vector<uint64_t> hs(b.sums.n);
        LDS_HIP(hipMemcpyAsync(hs.data(), b.sums.p, b.sums.bytes(), hipMemcpyDeviceToHost, s));
        LDS_HIP(hipStreamSynchronize(s));
        for (size_t j = 0; j < b.kernel_items.size(); ++j) {
            const int i = b.kernel_items[j];
            Graph& g = *b.gs[i];
            const int mode = b.modes[i];
            const SweepPlan& p = (mode == 2) ? g.edge_plan : g.tri_plan;
            if (p.nrows == 0) {
                std::vector<uint64_t> z((size_t)4 * b.iters[i], 0);
                fw_gap_from_sums(g.fw[mode == 2 ? 0 : 1], mode, b.iters[i], z.data());
            } else {
                fw_gap_from_sums(g.fw[mode == 2 ? 0 : 1], mode, b.iters[i], hs.data() + b.sum_off[j]);
            }
        }
    }
}

}  // namespace lds
