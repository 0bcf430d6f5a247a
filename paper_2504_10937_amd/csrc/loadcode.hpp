// 16-bit codes of the loads, by which the Frank-Wolfe sweep decides most
// comparisons of vertices without their 64-bit keys.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lds {

// the windows of an iteration's codes (see qcode), in one register: bases of
// the loads read and written, mantissa bits
struct Codes {
    uint32_t x;
    __host__ __device__ Codes(int in = 0, int out = 0, int mant = 11) : x((uint32_t)(in | (out << 8) | (mant << 16))) {}
    __host__ __device__ inline int in() const { return (int)(x & 255u); }
    __host__ __device__ inline int out() const { return (int)((x >> 8) & 255u); }
    __host__ __device__ inline int mant() const { return (int)(x >> 16); }
};

// Where the window begins, as the position of a leading one: that of D_i / 2 (a
// load of 1/2, an edge's even split) for edges and of D_i / 4 for triangles
// (1/3) and 4-cliques (1/4), so that the vertices of a lone pattern, whose
// loads come to lie about its even split, have codes of their own: a window
// from 1/2 on for every mode gave them all code 0, and each of their
// comparisons went to the keys (1M lone triangles 117 us a sweep, 57 now; 500k
// lone 4-cliques 131 and 41).  An octave lower for the 4-cliques would cut off
// the top: 190M clique slots, 52,120 at a vertex, 331 us from D_i / 2 on, 348
// from D_i / 8 on.
inline int code_octaves(int mode) { return mode == 2 ? 1 : 2; }  // below a load of 1 (D_i)
inline int code_base(int mode, uint64_t D) {
    const int b = 63 - __builtin_clzll(D) - code_octaves(mode);
    return b > 0 ? b : 0;
}

// 11 mantissa bits cover 32 octaves from there, any load; 12 cover 16 and are
// taken where no vertex has 2^16 patterns: its load is most / mode at the
// start and less later
inline int code_mant(int64_t most) { return most < (int64_t)1 << 16 ? 12 : 11; }

// 16-bit monotone code of a load numerator: a pseudo-float of `mant` mantissa
// bits whose exponents count from `base`, so the code is one of the load r =
// A / D_i and the same window of loads serves every iteration.  Numerators
// below it have code 0, those past it 65535.  A < A' implies qcode(A) <=
// qcode(A'), so different codes decide a comparison of packed keys exactly and
// equal codes fall back to the 64-bit keys.  The code array is a quarter of
// the key array, so the gathered working set stays in the L2 caches far more
// often.  A tie costs its batch a wait for the keys, and each bit halves them:
// 195M clique slots took 404 us with 10 bits and any exponent, 374 with 11 and
// 361 when ties were not looked up; 206M edge slots 822, 795 (12 bits) and 773.
__host__ __device__ inline uint16_t qcode(uint64_t A, int base, int mant) {
    const int z = __builtin_clzll(A | 1);  // (zero: below any window)
    const uint32_t top = (uint32_t)((A << z) >> 32) >> (31 - mant);  // leading one and mantissa
    const int c = ((62 - z - base) << mant) + (int)top;
    return (uint16_t)(c < 0 ? 0 : c > 65535 ? 65535 : c);
}

}  // namespace lds
