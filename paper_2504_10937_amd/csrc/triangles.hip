// Triangle listing for the triangle-density program (Eq. trcp, Alg. 6 use
// the triangle set T; the paper does not say how T is obtained), and
// 4-clique listing for the h-clique program that Eq. trcp generalises.
//
// Orientation: internal ids are sorted by degree (descending), so orienting
// every edge towards the smaller internal id points it at the endpoint of
// larger degree; out-lists N+(x) = {y in N(x) : y < x} are the prefixes of
// the ascending CSR rows and have length O(sqrt(m)).  A triangle with
// internal ids a > b > c is found exactly once, from the oriented edge
// (a -> b), as the element c of N+(a) ∩ N+(b).
//
// A wave takes up to 64 oriented edges of one vertex and looks up the shorter
// out-list of each edge's ends in the other (k_tri_units).  A count pass, an
// exclusive scan and a write pass give a deterministic order (oriented edges
// in CSR order, c ascending).
// The incidence CSR for the Frank-Wolfe pull sweep then holds, for every
// vertex with t_u > 0 (rows ordered by t_u descending), the other two
// vertices of each of its triangles, in triangle order.
#include <algorithm>

#include "graph.hpp"

namespace lds {

namespace {

constexpr int kT = 256;

__device__ inline int64_t lower_bound_i32(const int32_t* a, int64_t lo, int64_t hi, int32_t x) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// out-degree of every vertex: number of neighbours with a smaller internal id
__global__ void k_outdeg(const int64_t* rp, const int32_t* col, int64_t n, int32_t* outdeg) {
    const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (u >= n) return;
    outdeg[u] = (int32_t)(lower_bound_i32(col, rp[u], rp[u + 1], (int32_t)u) - rp[u]);
}

// The listing works in units: up to kUnitEdges consecutive oriented edges
// u -> v_i (v_i = N+(u)[i], i in [i0, i0 + kUnitEdges)) of one vertex, one
// wave each.  Edge i has candidates w: either all of N+(v_i) ("walk", looked up
// in N+(u)[0, i), staged in LDS) or all of N+(u)[0, i) ("probe", looked up in
// N+(v_i) in memory), both ascending, whichever is shorter up to the factor
// kProbeBias that a lookup in memory costs over one in LDS.  The candidates of
// a unit's edges are numbered consecutively and dealt to the lanes, so a wave
// is full whatever the list lengths, neighbouring lanes read neighbouring
// column entries, and ballots give the triangles in (edge, w) order.
// Bound: latency of the lookups.  One thread per slot of the CSR (both
// orientations, the row found by binary search, one list probed serially in
// the other) took 4.4 ms to count and 5.0 ms to write on 1M vertices, 2e7
// edges, 1.3e7 triangles; by units 1.2 and 1.5 ms.
constexpr int kUnitEdges = 64;
constexpr int kUnitList = 1024;  // entries of N+(u) staged per wave; longer lists are read from memory
constexpr int kProbeBias = 4;

__device__ inline int64_t unit_count(int32_t outdeg) {
    return outdeg < 2 ? 0 : (outdeg + kUnitEdges - 1) / kUnitEdges;
}

__global__ void k_unit_counts(const int32_t* outdeg, int64_t n, uint32_t* cnt) {
    const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (u < n) cnt[u] = (uint32_t)unit_count(outdeg[u]);
}

__global__ void k_unit_fill(const int32_t* outdeg, const uint64_t* first, int64_t n, int32_t* unit_u,
                            int32_t* unit_i0) {
    const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (u >= n) return;
    const int64_t c = unit_count(outdeg[u]), o = (int64_t)first[u];
    for (int64_t k = 0; k < c; ++k) {
        unit_u[o + k] = (int32_t)u;
        unit_i0[o + k] = (int32_t)(k * kUnitEdges);
    }
}

__device__ inline uint32_t wave_incl_scan_u32(uint32_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// count (WRITE = false: cnt per unit) or write (tri from off[unit], and the
// counts of the first two members: one atomic per unit for u, one per edge
// for v; the third members are counted by k_member_count)
template <bool WRITE>
__global__ __launch_bounds__(kT) void k_tri_units(const int64_t* rp, const int32_t* col, const int32_t* outdeg,
                                                  const int32_t* unit_u, const int32_t* unit_i0, int64_t units,
                                                  uint32_t* cnt, const uint64_t* off, int32_t* tri, int32_t* tc) {
    constexpr int NW = kT / 64;
    __shared__ int32_t list[NW][kUnitList];
    __shared__ uint32_t pre[NW][kUnitEdges];    // inclusive candidate counts of the unit's edges
    __shared__ uint32_t ecnt[NW][kUnitEdges];   // WRITE: triangles of each edge
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // whole waves; no workgroup barrier within
    for (int64_t k = (int64_t)blockIdx.x * NW + w; k < units; k += (int64_t)gridDim.x * NW) {
        __builtin_amdgcn_wave_barrier();  // the wave's LDS is rewritten by its next unit
        const int32_t u = unit_u[k];
        const int i0 = unit_i0[k];
        const int du = outdeg[u];
        const int64_t ua = rp[u];
        const int need = min(du, i0 + kUnitEdges);
        const bool staged = need <= kUnitList;
        const int i = i0 + lane;
        int32_t v = 0;
        int dv = 0;
        int64_t va = 0;
        if (i < du) {
            v = col[ua + i];
            dv = outdeg[v];
            va = rp[v];
        }
        if (staged)
            for (int q = lane; q < need; q += 64) list[w][q] = col[ua + q];
        const bool walk = (int64_t)dv <= (int64_t)kProbeBias * i;
        const uint32_t items = i < du && dv > 0 ? (uint32_t)(walk ? dv : i) : 0u;
        const uint32_t inc = wave_incl_scan_u32(items);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        pre[w][lane] = inc;
        if (WRITE) ecnt[w][lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t found = 0;
        uint64_t o = WRITE ? off[k] : 0;
        const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        for (uint32_t base = 0; base < total; base += 64) {
            const uint32_t c = base + (uint32_t)lane;
            const bool in = c < total;
            // the edge of candidate c: first e with pre[e] > c
            int e = 0;
#pragma unroll
            for (int st = 32; st > 0; st >>= 1)
                if (pre[w][e + st - 1] <= c) e += st;
            if (!in) e = 63;
            const int32_t ev = __shfl(v, e, 64);
            const int edv = __shfl(dv, e, 64);
            const int64_t eva = ((int64_t)__shfl((int)(va >> 32), e, 64) << 32) | (uint32_t)__shfl((int)(uint32_t)va, e, 64);
            const int ei = i0 + e;
            const uint32_t q = c - (e > 0 ? pre[w][e - 1] : 0u);
            bool hit = false;
            int32_t x = 0;
            if (in) {
                if ((int64_t)edv <= (int64_t)kProbeBias * ei) {  // walk N+(v), look up in N+(u)[0, ei)
                    x = col[eva + q];
                    if (staged) {
                        int lo = 0, hi = ei;
                        while (lo < hi) {
                            const int mid = (lo + hi) >> 1;
                            if (list[w][mid] < x) lo = mid + 1; else hi = mid;
                        }
                        hit = lo < ei && list[w][lo] == x;
                    } else {
                        const int64_t p = lower_bound_i32(col, ua, ua + ei, x);
                        hit = p < ua + ei && col[p] == x;
                    }
                } else {  // probe N+(u)[0, ei) in N+(v)
                    x = staged ? list[w][q] : col[ua + q];
                    const int64_t p = lower_bound_i32(col, eva, eva + edv, x);
                    hit = p < eva + edv && col[p] == x;
                }
            }
            const uint64_t H = __ballot(hit);
            if (WRITE) {
                if (hit) {
                    const uint64_t t = o + (uint64_t)__popcll(H & lt);
                    tri[3 * t + 0] = u;
                    tri[3 * t + 1] = ev;
                    tri[3 * t + 2] = x;
                    atomicAdd(&ecnt[w][e], 1u);
                }
                o += (uint64_t)__popcll(H);
            }
            found += (uint32_t)__popcll(H);
        }
        if (!WRITE) {
            if (lane == 0) cnt[k] = found;
            continue;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (ecnt[w][lane]) atomicAdd(&tc[v], (int32_t)ecnt[w][lane]);
        if (lane == 0 && found) atomicAdd(&tc[u], (int32_t)found);
    }
}

// Counts of a list of member ids (every stride-th entry of ids, from the
// first): patterns crowd on the vertices of smallest internal id, so the
// counts of the first nh ids are kept in an LDS histogram per workgroup
// (nearly the whole LDS of a CU) and added once at the end; the rest are
// atomics in memory.  Bound: atomic rate.  One atomic per member on the list
// in memory took 4.6 ms for 3.7e7 triangle members, and a histogram of 8192
// ids left 14 ms on 1.8e8 members of 4-cliques, whose blocks' vertices lie
// past it; this one takes 0.2 (for the 1.3e7 third members) and 0.8 ms.
constexpr int kCountIds = 36864;
constexpr int kCountT = 1024;
constexpr int64_t kCountPerWG = 16384;  // entries that are worth a workgroup's histogram
__global__ __launch_bounds__(kCountT) void k_member_count(const int32_t* ids, int64_t count, int stride, int nh,
                                                          int32_t* cnt) {
    extern __shared__ int32_t hist[];
    for (int i = threadIdx.x; i < nh; i += kCountT) hist[i] = 0;
    __syncthreads();
    const int64_t step = (int64_t)gridDim.x * kCountT;
    for (int64_t t0 = (int64_t)blockIdx.x * kCountT + threadIdx.x; t0 < count; t0 += 4 * step) {
        int32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = t0 + q * step < count ? ids[(t0 + q * step) * stride] : -1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (x[q] < 0) continue;
            if (x[q] < nh)
                atomicAdd(&hist[x[q]], 1);
            else
                atomicAdd(&cnt[x[q]], 1);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nh; i += kCountT)
        if (hist[i]) atomicAdd(&cnt[i], hist[i]);
}

void count_members(const int32_t* ids, int64_t count, int stride, int64_t n, int32_t* cnt, hipStream_t s) {
    if (count <= 0) return;
    const int nh = (int)std::min<int64_t>(n, kCountIds);
    LDS_HIP(hipFuncSetAttribute((const void*)k_member_count, hipFuncAttributeMaxDynamicSharedMemorySize,
                                kCountIds * (int)sizeof(int32_t)));
    const unsigned grid = std::min(grid_for(count, (int)kCountPerWG), kReduceWG);
    k_member_count<<<grid, kCountT, (size_t)nh * sizeof(int32_t), s>>>(ids, count, stride, nh, cnt);
    LDS_HIP(hipGetLastError());
}

__global__ void k_tmax(const int32_t* tc, int64_t n, int* out, unsigned long long* nz) {
    // grid-stride (the launch is capped at kReduceWG workgroups): one atomic
    // per wave on each of the two counters; with a wave per 64 entries the
    // waves of a 4M-entry array queued ~125k atomics on two addresses (0.75 ms)
    int d = 0;
    unsigned c = 0;  // entries > 0 (fewer than 2^32)
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
        const int x = tc[i];
        d = max(d, x);
        c += x > 0 ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) {
        d = max(d, __shfl_xor(d, off, 64));
        c += (unsigned)__shfl_xor((int)c, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(out, d);
        if (c) atomicAdd(nz, (unsigned long long)c);
    }
}

// rows: vertices with t > 0 ordered by t descending, internal id ascending
__global__ void k_row_keys(const int32_t* tc, int64_t n, int vb, int32_t tmax, uint64_t* keys) {
    const int64_t u = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (u >= n) return;
    // vertices without triangles sort last (key above every t > 0 key)
    const uint64_t t = (uint64_t)tc[u];
    keys[u] = ((t > 0 ? (uint64_t)(tmax - (int32_t)t) : (uint64_t)tmax) << vb) | (uint64_t)u;
}

__global__ void k_row_apply(const uint64_t* keys, int64_t nrows, int vb, const int32_t* tc, int32_t* rid,
                            int32_t* row_of, uint32_t* rcount) {
    const int64_t r = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (r >= nrows) return;
    const int32_t u = (int32_t)(keys[r] & ((1ull << vb) - 1));
    rid[r] = u;
    row_of[u] = (int32_t)r;
    rcount[r] = (uint32_t)tc[u];
}

template <int H>
__global__ void k_inc_keys(const int32_t* pat, int64_t np, const int32_t* row_of, int tb, uint64_t* keys) {
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t >= np) return;
    for (int j = 0; j < H; ++j) keys[H * t + j] = ((uint64_t)row_of[pat[H * t + j]] << tb) | (uint64_t)t;
}

// slot s: the other H-1 members of its pattern, in pattern order, and for
// triangles the pattern
template <int H, bool PACKED>
__global__ void k_inc_pay(const uint64_t* keys, int64_t ns, int tb, const int32_t* pat, const int32_t* rid,
                          int32_t* pay, int32_t* tos) {
    const int64_t s = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (s >= ns) return;
    const uint64_t k = keys[s];
    const int64_t t = (int64_t)(k & ((1ull << tb) - 1));
    const int32_t x = rid[k >> tb];
    if (PACKED) {
        const int4 y = reinterpret_cast<const int4*>(pat)[t];
        const bool i0 = y.x == x, i1 = i0 || y.y == x, i2 = i1 || y.z == x;  // x found by then
        const uint64_t a = (uint32_t)(i0 ? y.y : y.x), b = (uint32_t)(i1 ? y.z : y.y), c = (uint32_t)(i2 ? y.w : y.z);
        reinterpret_cast<uint64_t*>(pay)[s] = a | (b << PackedSlot::kBits) | (c << (2 * PackedSlot::kBits));
        return;
    }
    int o = 0;
    for (int j = 0; j < H; ++j) {
        const int32_t y = pat[H * t + j];
        if (y != x) pay[(H - 1) * s + o++] = y;
    }
    if (H == 3) tos[s] = (int32_t)t;
}

__global__ void k_set_last(int64_t* rowptr, int64_t idx, const uint64_t* total) { rowptr[idx] = (int64_t)*total; }

// 4-cliques: a clique with internal ids a > b > c > d is found exactly once,
// from its triangle (a, b, c): (a, b, d) is a triangle too, and the triangles
// are in the order of (a, b, c), so the candidates d are the third members of
// the triangles of (a, b) before this one, and d is confirmed by one search,
// in N+(c).  One thread per triangle walks them downwards, galloping down
// N+(c) as d falls.  When they are many against N+(c), it walks N+(c) instead
// and searches N+(a) and N+(b).  A count pass, a scan and a write pass (from
// each triangle's last place down) give the order: triangle order, d
// ascending.  Bound: the chain of dependent reads of a search.  On 49M cliques
// the passes take 1.26 and 1.83 ms; walking the shortest of the three
// out-lists and searching the other two took 2.43 and 3.15.
template <bool WRITE>
__global__ void k_clique_tris(const int64_t* rp, const int32_t* col, const int32_t* tri, int64_t T, uint32_t* cnt,
                              const uint64_t* off, int32_t* q4) {
    const int64_t t = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (t >= T) return;
    if (WRITE && cnt[t] == 0) return;
    const int32_t a = tri[3 * t], b = tri[3 * t + 1], c = tri[3 * t + 2];  // a > b > c
    const int64_t lo = rp[c];
    int64_t end = lower_bound_i32(col, lo, rp[c + 1], c);  // N+(c) is [lo, end)
    const int64_t limit = 2 * (end - lo) + 16;
    uint64_t o = WRITE ? off[t] + cnt[t] : 0;
    uint32_t k = 0;
    auto found = [&](int32_t d) {
        if (WRITE) reinterpret_cast<int4*>(q4)[--o] = make_int4(a, b, c, d);
        ++k;
    };
    int64_t p = end;  // the members of N+(c) from p on are above every candidate left
    int64_t i = t - 1;
    for (; i >= 0 && p > lo && t - i <= limit; --i) {
        if (tri[3 * i] != a || tri[3 * i + 1] != b) break;
        const int32_t d = tri[3 * i + 2];
        // the first member >= d lies in (p - step, p]
        int64_t step = 1;
        while (p - step >= lo && col[p - step] >= d) step <<= 1;
        p = lower_bound_i32(col, max(lo, p - step), p - (step >> 1), d);
        if (p < end && col[p] == d) found(d);
    }
    if (i >= 0 && p > lo && t - i > limit) {  // the rest of N+(c), downwards
        int64_t pa = rp[a], ea = lower_bound_i32(col, pa, rp[a + 1], c);
        int64_t pb = rp[b], eb = lower_bound_i32(col, pb, rp[b + 1], c);
        while (--p >= lo) {
            const int32_t d = col[p];
            ea = lower_bound_i32(col, pa, ea, d + 1);  // N(a) up to d
            if (ea == pa) break;
            if (col[ea - 1] != d) continue;
            eb = lower_bound_i32(col, pb, eb, d + 1);
            if (eb == pb) break;
            if (col[eb - 1] == d) found(d);
        }
    }
    if (!WRITE) cnt[t] = k;
}

template <class T>
T d2h(const T* p, hipStream_t s) {
    T v;
    LDS_HIP(hipMemcpyAsync(&v, p, sizeof(T), hipMemcpyDeviceToHost, s));
    LDS_HIP(hipStreamSynchronize(s));
    return v;
}

// Incidence CSR of a pattern list (H vertices per pattern) for the pull
// sweep: rows are the vertices with count > 0 ordered by count descending
// (internal id ascending), each row holding, for every pattern at the
// vertex, the other H-1 members (in pattern order), patterns in list order.
template <int H>
void build_incidence_plan(Graph& g, const int32_t* pat, int64_t np, const int32_t* count, SweepPlan& p,
                          int64_t& cmax, hipStream_t s) {
    const int64_t n = g.n;
    LDS_CHECK(np < (int64_t)INT32_MAX, ST_OVERFLOW, "too many patterns for 32-bit pattern indices");
    p.h = H;
    DBuf<int> tmax;
    DBuf<unsigned long long> nz;
    tmax.alloc(1, s);
    nz.alloc(1, s);
    LDS_HIP(hipMemsetAsync(tmax.p, 0, sizeof(int), s));
    LDS_HIP(hipMemsetAsync(nz.p, 0, sizeof(unsigned long long), s));
    if (n > 0) {
        k_tmax<<<std::min(grid_for(n, kT), kReduceWG), kT, 0, s>>>(count, n, tmax.p, nz.p);
        LDS_HIP(hipGetLastError());
    }
    cmax = d2h(tmax.p, s);
    const int64_t nrows = (int64_t)d2h(nz.p, s);
    p.nrows = nrows;
    p.nslots = H * np;
    p.own_rid.alloc(nrows, s);
    p.own_rp.alloc(nrows + 1, s);
    p.packed = H == 4 && n <= PackedSlot::kMaxVertices;
    p.own_py.alloc((p.packed ? 2 : H - 1) * H * np, s);
    DBuf<int32_t>& row_of = p.own_row_of;
    row_of.alloc(n, s);
    if (n) LDS_HIP(hipMemsetAsync(row_of.p, 0xff, n * sizeof(int32_t), s));  // -1: no pattern
    DBuf<uint32_t> rcount;
    rcount.alloc(nrows, s);
    if (nrows > 0) {
        const int vb = g.vbits;
        DBuf<uint64_t> rk, rt;
        rk.alloc(n, s);
        rt.alloc(n, s);
        k_row_keys<<<grid_for(n, kT), kT, 0, s>>>(count, n, vb, (int32_t)cmax, rk.p);
        LDS_HIP(hipGetLastError());
        // keys in id order: the stable sort needs the count bits only
        radix_sort_u64(rk, nullptr, n, vb, vb + bits_for((uint64_t)cmax), rt, nullptr, s);
        k_row_apply<<<grid_for(nrows, kT), kT, 0, s>>>(rk.p, nrows, vb, count, p.own_rid.p, row_of.p, rcount.p);
        LDS_HIP(hipGetLastError());
    }
    DBuf<uint64_t> tot;
    tot.alloc(1, s);
    exclusive_scan_u32_to_u64(rcount.p, (uint64_t*)p.own_rp.p, nrows, tot.p, s);
    k_set_last<<<1, 1, 0, s>>>(p.own_rp.p, nrows, tot.p);
    LDS_HIP(hipGetLastError());
    if (np > 0) {
        const int tb = bits_for((uint64_t)(np - 1)) > 0 ? bits_for((uint64_t)(np - 1)) : 1;
        const int rb = bits_for((uint64_t)nrows);
        LDS_CHECK(tb + rb <= 64, ST_OVERFLOW, "pattern incidence key exceeds 64 bits");
        DBuf<uint64_t> ik, it;
        ik.alloc(H * np, s);
        it.alloc(H * np, s);
        k_inc_keys<H><<<grid_for(np, kT), kT, 0, s>>>(pat, np, row_of.p, tb, ik.p);
        LDS_HIP(hipGetLastError());
        // the keys are made in pattern order and the sort is stable, so the
        // row bits alone order them
        radix_sort_u64(ik, nullptr, H * np, tb, tb + rb, it, nullptr, s);
        if (H == 3) p.own_tos.alloc(H * np, s);
        if (p.packed)
            k_inc_pay<H, H == 4><<<grid_for(H * np, kT), kT, 0, s>>>(ik.p, H * np, tb, pat, p.own_rid.p, p.own_py.p,
                                                                   nullptr);
        else
            k_inc_pay<H, false><<<grid_for(H * np, kT), kT, 0, s>>>(ik.p, H * np, tb, pat, p.own_rid.p, p.own_py.p,
                                                                  p.own_tos.p);
        LDS_HIP(hipGetLastError());
    }
    p.rid = p.own_rid.p;
    p.rp = p.own_rp.p;
    p.py = p.own_py.p;
    build_sweep_plan(p, s);
}

}  // namespace

namespace {
// triangles at each vertex, from the incidence rows (a row's slots are in
// ascending triangle order, so each list is too)
__global__ void k_vtx_tcount(const int32_t* row_of, const int64_t* rp, int64_t n, uint64_t* cnt) {
    const int64_t v = (int64_t)blockIdx.x * kT + threadIdx.x;
    if (v >= n) return;
    const int32_t r = row_of[v];
    cnt[v] = r < 0 ? 0 : (uint64_t)(rp[r + 1] - rp[r]);
}

__global__ void k_vtx_tfill(const int32_t* rid, const int64_t* rp, int64_t nrows, const int32_t* tos,
                            const uint64_t* off, int32_t* tinc) {
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (kT / 64) + (threadIdx.x >> 6);
    if (r >= nrows) return;
    const int64_t base = (int64_t)off[rid[r]] - rp[r];
    for (int64_t q = rp[r] + lane; q < rp[r + 1]; q += 64) tinc[base + q] = tos[q];
}
}  // namespace

void vertex_triangle_lists(const Graph& g, int64_t* trp_host, int32_t* tinc_host, hipStream_t s) {
    const int64_t n = g.n;
    LDS_CHECK(g.T >= 0, ST_INVALID, "triangles are not listed");
    if (n == 0) return;
    const SweepPlan& p = g.tri_plan;
    DBuf<uint64_t> off;
    off.alloc(n + 1, s);
    k_vtx_tcount<<<grid_for(n, kT), kT, 0, s>>>(p.own_row_of.p, p.rp, n, off.p);
    LDS_HIP(hipGetLastError());
    exclusive_scan_u64(off.p, off.p, n, off.p + n, s);
    DBuf<int32_t> tinc;
    tinc.alloc(3 * g.T, s);
    if (g.T > 0 && p.nrows > 0) {
        k_vtx_tfill<<<grid_for(p.nrows, kT / 64), kT, 0, s>>>(p.rid, p.rp, p.nrows, p.own_tos.p, off.p, tinc.p);
        LDS_HIP(hipGetLastError());
    }
    LDS_HIP(hipMemcpyAsync(trp_host, off.p, (n + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (g.T > 0) LDS_HIP(hipMemcpyAsync(tinc_host, tinc.p, 3 * g.T * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    LDS_HIP(hipStreamSynchronize(s));
}

void list_triangles(Graph& g, hipStream_t s) {
    const int64_t n = g.n, ns = 2 * g.m;
    sort_rows(g, s);
    g.tcount.alloc(n, s);
    if (n) LDS_HIP(hipMemsetAsync(g.tcount.p, 0, n * sizeof(int32_t), s));
    int64_t T = 0;
    if (ns > 0) {
        DBuf<int32_t> outdeg;
        outdeg.alloc(n, s);
        k_outdeg<<<grid_for(n, kT), kT, 0, s>>>(g.rowptr.p, g.col.p, n, outdeg.p);
        LDS_HIP(hipGetLastError());
        // units of work: kUnitEdges oriented edges of one vertex each
        DBuf<uint32_t> cnt;
        DBuf<uint64_t> off, tot;
        cnt.alloc(n, s);
        off.alloc(n, s);
        tot.alloc(1, s);
        k_unit_counts<<<grid_for(n, kT), kT, 0, s>>>(outdeg.p, n, cnt.p);
        LDS_HIP(hipGetLastError());
        exclusive_scan_u32_to_u64(cnt.p, off.p, n, tot.p, s);
        const int64_t units = (int64_t)d2h(tot.p, s);
        if (units > 0) {
            DBuf<int32_t> unit_u, unit_i0;
            unit_u.alloc(units, s);
            unit_i0.alloc(units, s);
            k_unit_fill<<<grid_for(n, kT), kT, 0, s>>>(outdeg.p, off.p, n, unit_u.p, unit_i0.p);
            LDS_HIP(hipGetLastError());
            cnt.alloc(units, s);
            off.alloc(units, s);
            const unsigned grid = stride_grid(units, kT / 64);
            k_tri_units<false><<<grid, kT, 0, s>>>(g.rowptr.p, g.col.p, outdeg.p, unit_u.p, unit_i0.p, units, cnt.p,
                                                   nullptr, nullptr, nullptr);
            LDS_HIP(hipGetLastError());
            exclusive_scan_u32_to_u64(cnt.p, off.p, units, tot.p, s);
            T = (int64_t)d2h(tot.p, s);
            g.tri.alloc(3 * T, s);
            if (T > 0) {
                k_tri_units<true><<<grid, kT, 0, s>>>(g.rowptr.p, g.col.p, outdeg.p, unit_u.p, unit_i0.p, units,
                                                      nullptr, off.p, g.tri.p, g.tcount.p);
                LDS_HIP(hipGetLastError());
                count_members(g.tri.p + 2, T, 3, n, g.tcount.p, s);
            }
        }
    }
    g.T = T;
    build_incidence_plan<3>(g, g.tri.p, T, g.tcount.p, g.tri_plan, g.t_max, s);
}

void list_cliques4(Graph& g, hipStream_t s) {
    if (g.T < 0) list_triangles(g, s);  // also sorts the rows
    const int64_t n = g.n, T = g.T;
    g.qcount.alloc(n, s);
    if (n) LDS_HIP(hipMemsetAsync(g.qcount.p, 0, n * sizeof(int32_t), s));
    int64_t Q = 0;
    if (T > 0) {
        DBuf<uint32_t> cnt;
        DBuf<uint64_t> off, tot;
        cnt.alloc(T, s);
        off.alloc(T, s);
        tot.alloc(1, s);
        k_clique_tris<false><<<grid_for(T, kT), kT, 0, s>>>(g.rowptr.p, g.col.p, g.tri.p, T, cnt.p, nullptr, nullptr);
        LDS_HIP(hipGetLastError());
        exclusive_scan_u32_to_u64(cnt.p, off.p, T, tot.p, s);
        Q = (int64_t)d2h(tot.p, s);
        g.q4.alloc(4 * Q, s);
        if (Q > 0) {
            k_clique_tris<true><<<grid_for(T, kT), kT, 0, s>>>(g.rowptr.p, g.col.p, g.tri.p, T, cnt.p, off.p, g.q4.p);
            LDS_HIP(hipGetLastError());
            count_members(g.q4.p, 4 * Q, 1, n, g.qcount.p, s);
        }
    }
    g.Q4 = Q;
    build_incidence_plan<4>(g, g.q4.p, Q, g.qcount.p, g.clique_plan, g.q_max, s);
}

}  // namespace lds
