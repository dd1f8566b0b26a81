// A probe vector v[a d_B + b] into the contraction operand Xt (row (k, b),
// reduction index a), through LDS tiles: the vector is read once along b, the
// operand written in whole 16-byte units along a.  The plain form, one entry
// per thread, read each entry at a stride of d_B as well and stored 2-byte
// pieces: for 8 vectors of 2^20 entries in split BF16 the recurrence's last
// pass took 145 us with it and 82 with tiles (60 to 48 bytes per entry).
#pragma once
#include "operands.h"

namespace tnslq {

// a tile: up to 32 b by 64 a, or up to 256 entries where d_B is below 4 (the
// explicit operator's vectors have d_B = 1); whole units of a
constexpr int XT_TA = 64, XT_TB = 32;
__host__ __device__ inline int xt_tb(int64_t dB) { return (int)(dB < XT_TB ? dB : XT_TB); }
__host__ __device__ inline int xt_ta(int64_t dA, int64_t dB) {
    const int t = dB < 4 ? 256 / (int)dB / 8 * 8 : XT_TA;
    return (int)(dA < t ? dA : t);
}
__host__ __device__ inline int64_t xt_tiles(int64_t dA, int64_t dB) {
    return ((dA + xt_ta(dA, dB) - 1) / xt_ta(dA, dB)) * ((dB + xt_tb(dB) - 1) / xt_tb(dB));
}

// Called by whole blocks of 256 threads.  f(v) is stored; keep(e, f(v)) sees
// every entry e = a d_B + b once.
template <int PREC, typename F, typename G>
__device__ inline void vector_to_xt(const double2 *__restrict__ v, void *__restrict__ Xt, int64_t xt_nst, int64_t k,
                                    int64_t dA, int64_t dB, F f, G keep) {
    constexpr int EPU = brick_epu(PREC);
    __shared__ double2 tile[XT_TA * XT_TB];
    const int ta = xt_ta(dA, dB), tb = xt_tb(dB);
    const int64_t ntb = (dB + tb - 1) / tb, tiles = xt_tiles(dA, dB);
    for (int64_t tl = blockIdx.x; tl < tiles; tl += gridDim.x) {
        const int64_t a0 = (tl / ntb) * ta, b0 = (tl % ntb) * tb;
        for (int i = threadIdx.x; i < ta * tb; i += 256) {
            const int64_t a = a0 + i / tb, b = b0 + i % tb;
            double2 x = make_double2(0.0, 0.0);
            if (a < dA && b < dB) {
                const int64_t e = a * dB + b;
                x = f(v[e]);
                keep(e, x);
            }
            tile[i] = x;
        }
        __syncthreads();
        const int nu = (ta + EPU - 1) / EPU;
        for (int i = threadIdx.x; i < nu * tb; i += 256) {
            const int bl = i % tb, al = i / tb * EPU;
            if (b0 + bl < dB && a0 + al < dA) {
                double2 u[EPU];
#pragma unroll
                for (int t = 0; t < EPU; ++t)
                    u[t] = al + t < ta ? tile[(al + t) * tb + bl] : make_double2(0.0, 0.0);
                store_unit<PREC>(Xt, brick_index(PREC, xt_nst, k * dB + b0 + bl, a0 + al), u);
            }
        }
        __syncthreads();
    }
}

}  // namespace tnslq
