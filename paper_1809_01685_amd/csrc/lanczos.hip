// FP64 Lanczos recurrence, reorthogonalisation, Gauss quadrature and
// Hutchinson statistics (Sec. III, Algorithm 1; Sec. VIII).
//
// Vectors are complex128, one row of d_A d_B elements per probe.  Reductions
// over a vector are done in two fixed-order stages (per-block tree, then a
// sequential sum of the block partials) so that results are bitwise
// reproducible run to run; no floating-point atomics are used.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "breakdown.h"
#include "tnslq_internal.h"
#include "wave.h"
#include "xt_tile.h"

namespace tnslq {
namespace {

// Fixed-order sum over a 256-thread block (each wave's in registers, then LDS:
// with shuffles through LDS, twelve in a row, and the scans of the breakdown test
// likewise, passA, passB and passC at n = 4096 took 7.5, 11.4 and 6.3 us instead
// of 6.6, 10.5 and 5.5).
__device__ inline double block_sum(double v, double *sh) {
    v = wave_tree_total(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0) {
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
        sh[8] = t;
    }
    __syncthreads();
    return sh[8];
}

// The same sum where one thread of the block needs it (thread 0): one barrier,
// with LDS of its own.
__device__ inline double block_sum_first(double v, double (&sh)[4]) {
    v = wave_tree_total(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
    return t;
}

// Sum of partials[0..cnt) in a fixed order, the same in every block.  Up to 64
// of them every wave adds for itself.
__device__ inline double sum_partials(const double *p, int cnt, double *sh) {
    const int lane = threadIdx.x & 63;
    if (cnt <= 64) return 0.0 + wave_tree_total(lane < cnt ? p[lane] : 0.0);
    double v = 0.0;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) v += p[i];
    return block_sum(v, sh);
}

__device__ inline void elem_range(int64_t n, int nblk, int64_t &beg, int64_t &end) {
    const int64_t chunk = (n + nblk - 1) / nblk;
    beg = (int64_t)blockIdx.x * chunk;
    end = beg + chunk < n ? beg + chunk : n;
}

// w = Y - beta_j q_{j-1} with Y the sum of the contraction's split partials;
// partial sums of Re<q_j, w>.
template <typename AccT>
__global__ void __launch_bounds__(256) k_passA(const AccT *__restrict__ part, int S, int64_t split_stride,
                                               int k0, int64_t n, const double2 *__restrict__ q_prev,
                                               const double2 *__restrict__ q_cur, double2 *__restrict__ w,
                                               const double *__restrict__ alpha,
                                               const double *__restrict__ beta, int m, int j, int nblk,
                                               double *__restrict__ dotpart, uint64_t *start) {
    __shared__ double sh[4];
    stamp(start);
    const int kl = blockIdx.y, k = k0 + kl;
    const double *ak = alpha + (int64_t)k * m;
    const double *bk = beta + (int64_t)k * (m + 1);
    const bool live = first_break(ak, bk, j - 1) == 0;
    const double bj = (j > 1) ? bk[j - 1] : 0.0;
    int64_t beg, end;
    elem_range(n, nblk, beg, end);
    double acc = 0.0;
    const int64_t base = (int64_t)k * n;
    for (int64_t e = beg + threadIdx.x; e < end; e += blockDim.x) {
        double re = 0.0, im = 0.0;
        for (int s = 0; s < S; ++s) {
            AccT v = part[s * split_stride + (int64_t)kl * n + e];
            re += (double)v.x;
            im += (double)v.y;
        }
        if (j > 1) {
            double2 p = q_prev[base + e];
            re -= bj * p.x;
            im -= bj * p.y;
        }
        if (!live) re = im = 0.0;
        w[base + e] = make_double2(re, im);
        double2 q = q_cur[base + e];
        acc += q.x * re + q.y * im;
    }
    acc = block_sum_first(acc, sh);
    if (threadIdx.x == 0) dotpart[(int64_t)k * nblk + blockIdx.x] = acc;
}

// alpha_j = Re<q_j, w>;  w -= alpha_j q_j;  partial sums of |w|^2.
__global__ void __launch_bounds__(256) k_passB(const double *__restrict__ dotpart, int64_t n,
                                               const double2 *__restrict__ q_cur, double2 *__restrict__ w,
                                               double *__restrict__ alpha, const double *__restrict__ beta,
                                               int m, int j, int nblk, double *__restrict__ nrmpart,
                                               uint64_t *start) {
    __shared__ double sh[16], sh1[4];
    stamp(start);
    const int k = blockIdx.y;
    const double *ak = alpha + (int64_t)k * m;
    const double *bk = beta + (int64_t)k * (m + 1);
    const bool live = first_break(ak, bk, j - 1) == 0;
    double a = sum_partials(dotpart + (int64_t)k * nblk, nblk, sh);
    if (!live) a = 0.0;
    int64_t beg, end;
    elem_range(n, nblk, beg, end);
    const int64_t base = (int64_t)k * n;
    double acc = 0.0;
    for (int64_t e = beg + threadIdx.x; e < end; e += blockDim.x) {
        double2 q = q_cur[base + e], v = w[base + e];
        v.x -= a * q.x;
        v.y -= a * q.y;
        w[base + e] = v;
        acc += v.x * v.x + v.y * v.y;
    }
    acc = block_sum_first(acc, sh1);
    if (threadIdx.x == 0) nrmpart[(int64_t)k * nblk + blockIdx.x] = acc;
    if (blockIdx.x == 0 && threadIdx.x == 0) alpha[(int64_t)k * m + (j - 1)] = a;
}

// Classical Gram-Schmidt, twice, against the nvec stored vectors Q_i of the
// probe.  It is bound by reading Q (nvec times the vector), so the recurrence
// reads it three times instead of four: the kernels that change w also take
// the next dot products of the chunk they hold, the second of them on the
// chunk of Q just read, from cache.  A block holds a chunk of blockDim.x
// elements of w, one per thread; for the dot products it leaves the chunk in
// LDS and each wave takes every fourth (second, only) vector, so that one
// wave sum ends a vector instead of two block sums.  Chunks are small (256
// elements, down to 64 where the block count would leave the chip idle), so
// that the chunks of Q in flight stay in cache between the two uses.  40 steps
// of 32 probes: 28.1 to 21.2 ms at n = 65536 (4.4 TB/s of Q read), 4.24 to
// 1.48 ms at n = 4096, where the block sums were most of the time.
__device__ inline void chunk_dots(const double2 *__restrict__ Q, int nvec, int64_t slot, int64_t at, int cnt,
                                  const double2 *ws, int nchunk, double2 *__restrict__ hpart) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    constexpr int VU = 2;   // vectors in flight per wave
    double2 v[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] = lane + 64 * x < cnt ? ws[lane + 64 * x] : make_double2(0.0, 0.0);
    for (int i0 = wid; i0 < nvec; i0 += VU * nw) {
        double2 q[VU][4];
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int i = i0 + u * nw;
            const double2 *qi = Q + (int64_t)i * slot + at;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                q[u][x] = i < nvec && lane + 64 * x < cnt ? qi[lane + 64 * x] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < VU; ++u) {
            const int i = i0 + u * nw;
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                re += q[u][x].x * v[x].x + q[u][x].y * v[x].y;   // conj(q) * v
                im += q[u][x].x * v[x].y - q[u][x].y * v[x].x;
            }
            re = wave_total(re);
            im = wave_total(im);
            if (lane == 0 && i < nvec) hpart[(int64_t)i * nchunk] = make_double2(re, im);
        }
    }
}

// v -= sum_i h_i Q_i of one element
__device__ inline void remove_vectors(const double2 *__restrict__ Qe, int nvec, int64_t slot, const double2 *hs,
                                      double2 &v) {
#pragma unroll 8
    for (int i = 0; i < nvec; ++i) {
        const double2 q = Qe[(int64_t)i * slot], c = hs[i];
        v.x -= c.x * q.x - c.y * q.y;
        v.y -= c.x * q.y + c.y * q.x;
    }
}

// The probe's h_i into LDS: from h, or, with few chunks, from their partial
// sums
__device__ inline void load_h(int k, int nvec, int nchunk, const double2 *__restrict__ hpart,
                              const double2 *__restrict__ h, double2 *hs) {
    for (int i = threadIdx.x; i < nvec; i += blockDim.x) {
        double2 s = make_double2(0.0, 0.0);
        if (nchunk > REORTH_FOLD) {
            s = h[(int64_t)k * nvec + i];
        } else {
            const double2 *p = hpart + ((int64_t)k * nvec + i) * nchunk;
#pragma unroll 8
            for (int b = 0; b < nchunk; ++b) {
                s.x += p[b].x;
                s.y += p[b].y;
            }
        }
        hs[i] = s;
    }
    __syncthreads();
}

// passB of a reorthogonalised step: alpha_j, w -= alpha_j q_j, and the first
// dot products.
__global__ void __launch_bounds__(256) k_passB_dots(const double *__restrict__ dotpart, int nblk, int64_t n,
                                                    const double2 *__restrict__ Q, int64_t slot,
                                                    double2 *__restrict__ w, double *__restrict__ alpha,
                                                    const double *__restrict__ beta, int m, int j, int nchunk,
                                                    double2 *__restrict__ hpart, uint64_t *start) {
    __shared__ double sh[16];
    __shared__ double2 ws[256];
    stamp(start);
    const int k = blockIdx.y;
    const bool live = first_break(alpha + (int64_t)k * m, beta + (int64_t)k * (m + 1), j - 1) == 0;
    double a = sum_partials(dotpart + (int64_t)k * nblk, nblk, sh);
    if (!live) a = 0.0;
    const int64_t beg = (int64_t)blockIdx.x * blockDim.x, at = (int64_t)k * n + beg;
    const int cnt = (int)(n - beg < (int64_t)blockDim.x ? n - beg : (int64_t)blockDim.x);
    if ((int)threadIdx.x < cnt) {
        const double2 q = Q[(int64_t)(j - 1) * slot + at + threadIdx.x];
        double2 v = w[at + threadIdx.x];
        v.x -= a * q.x;
        v.y -= a * q.y;
        w[at + threadIdx.x] = v;
        ws[threadIdx.x] = v;
    }
    __syncthreads();
    chunk_dots(Q, j, slot, at, cnt, ws, nchunk, hpart + (int64_t)k * j * nchunk + blockIdx.x);
    if (blockIdx.x == 0 && threadIdx.x == 0) alpha[(int64_t)k * m + (j - 1)] = a;
}

// w -= sum_i h_i Q_i and the second dot products.
__global__ void __launch_bounds__(256) k_reorth_update_dots(const double2 *__restrict__ Q, int nvec, int64_t slot,
                                                            int64_t n, const double2 *__restrict__ h,
                                                            const double2 *__restrict__ hpart_in,
                                                            double2 *__restrict__ w, int nchunk,
                                                            double2 *__restrict__ hpart) {
    __shared__ double2 ws[256];
    __shared__ double2 hs[TNSLQ_MAX_STEPS + 1];
    const int k = blockIdx.y;
    load_h(k, nvec, nchunk, hpart_in, h, hs);
    const int64_t beg = (int64_t)blockIdx.x * blockDim.x, at = (int64_t)k * n + beg;
    const int cnt = (int)(n - beg < (int64_t)blockDim.x ? n - beg : (int64_t)blockDim.x);
    if ((int)threadIdx.x < cnt) {
        double2 v = w[at + threadIdx.x];
        remove_vectors(Q + at + threadIdx.x, nvec, slot, hs, v);
        w[at + threadIdx.x] = v;
        ws[threadIdx.x] = v;
    }
    __syncthreads();
    chunk_dots(Q, nvec, slot, at, cnt, ws, nchunk, hpart + (int64_t)k * nvec * nchunk + blockIdx.x);
}

// h_i = the sum of the chunks' partial sums, one wave per (probe, i).
__global__ void __launch_bounds__(256) k_reorth_reduce(const double2 *__restrict__ hpart, int nvec, int nchunk,
                                                       double2 *__restrict__ h) {
    const int k = blockIdx.y, lane = threadIdx.x & 63, i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= nvec) return;
    const double2 *p = hpart + ((int64_t)k * nvec + i) * nchunk;
    double re = 0.0, im = 0.0;
    for (int b = lane; b < nchunk; b += 64) {
        re += p[b].x;
        im += p[b].y;
    }
    re = wave_total(re);
    im = wave_total(im);
    if (lane == 0) h[(int64_t)k * nvec + i] = make_double2(re, im);
}

// w -= sum_i h_i Q_i and the partial sums of |w|^2, over the recurrence's own
// blocks.
__global__ void __launch_bounds__(256) k_reorth_update(const double2 *__restrict__ Q, int nvec, int64_t slot,
                                                       int64_t n, const double2 *__restrict__ h,
                                                       const double2 *__restrict__ hpart, int nchunk,
                                                       double2 *__restrict__ w, int nblk,
                                                       double *__restrict__ nrmpart) {
    __shared__ double sh[4];
    __shared__ double2 hs[TNSLQ_MAX_STEPS + 1];
    const int k = blockIdx.y;
    load_h(k, nvec, nchunk, hpart, h, hs);
    int64_t beg, end;
    elem_range(n, nblk, beg, end);
    const int64_t base = (int64_t)k * n;
    double acc = 0.0;
    for (int64_t e = beg + threadIdx.x; e < end; e += blockDim.x) {
        double2 v = w[base + e];
        remove_vectors(Q + base + e, nvec, slot, hs, v);
        w[base + e] = v;
        acc += v.x * v.x + v.y * v.y;
    }
    acc = block_sum_first(acc, sh);
    if (threadIdx.x == 0) nrmpart[(int64_t)k * nblk + blockIdx.x] = acc;
}

// beta_{j+1} = ||w||, breakdown test, q_{j+1} = w / beta_{j+1} (0 after a
// breakdown), and the transposed low-precision copy for the next contraction.
template <int PREC>
__global__ void __launch_bounds__(256) k_passC(const double *__restrict__ nrmpart, int64_t n, int64_t dA,
                                               int64_t dB, const double2 *__restrict__ w,
                                               double2 *__restrict__ q_next, void *__restrict__ Xt,
                                               int64_t xt_nst, const double *__restrict__ alpha,
                                               double *__restrict__ beta, int m, int j, int nblk) {
    __shared__ double sh[16];
    const int k = blockIdx.y;
    const double *ak = alpha + (int64_t)k * m;
    double *bk = beta + (int64_t)k * (m + 1);
    double amax, bmax;
    const bool live = first_break(ak, bk, j - 1, amax, bmax) == 0;
    double b = sqrt(sum_partials(nrmpart + (int64_t)k * nblk, nblk, sh));
    if (!live) b = 0.0;
    amax = fmax(amax, fabs(ak[j - 1]));
    if (j >= 2) bmax = fmax(bmax, bk[j - 1]);
    const bool cont = live && !(b <= BREAKDOWN_TOL * (amax + bmax));
    const double2 *wk = w + (int64_t)k * n;
    double2 *qk = q_next + (int64_t)k * n;
    auto unit = [&](double2 v) { return cont ? make_double2(v.x / b, v.y / b) : make_double2(0.0, 0.0); };
    if (Xt) {
        vector_to_xt<PREC>(wk, Xt, xt_nst, k, dA, dB, unit, [&](int64_t e, double2 q) { qk[e] = q; });
    } else {
        const int64_t gstride = (int64_t)gridDim.x * blockDim.x;
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gstride) qk[e] = unit(wk[e]);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) bk[j] = b;
}

__global__ void __launch_bounds__(64) k_steps(const double *__restrict__ alpha, const double *__restrict__ beta, int m,
                                              int jdone, int *__restrict__ steps, uint64_t *start) {
    if (start && *start == 0) stamp(start);   // the step's first check is its end
    const int k = blockIdx.x;
    const int s = first_break(alpha + (int64_t)k * m, beta + (int64_t)k * (m + 1), jdone);
    if (threadIdx.x == 0) steps[k] = s ? s : jdone;
}

// Eigenvalues and first eigenvector components of the symmetric tridiagonal
// (d, e) by implicit QL with Wilkinson-type shifts (Bowdler, Martin, Reinsch
// & Wilkinson 1968), accumulating only the first row of the eigenvector
// matrix, by one wave: entry i lives in lane i % 64 of register i / 64.  e[i]
// couples d[i] and d[i+1]; e[n-1] must be 0.  On return d holds the
// eigenvalues and z the first components.  The rotations are one serial
// chain, so the wave carries its state (g, s, c, p and the entries i + 1 of d
// and z) uniformly, reads entry i by a lane read and writes entry i + 1 by a
// lane select; the search for a negligible e is one ballot.  Rotations walk the
// registers one after the other (picking one by the index in every rotation, 4096
// probes of 100 steps took 217 ms, where one thread per problem took 206: 168 now).
// Magnitudes must be scaled to about 1 (the squares of a rotation are taken as they are).
template <int R>
struct LaneVec {
    double v[R];
    __device__ inline double get(int i) const {
        if constexpr (R == 1) return lane_value(v[0], i);
        return i < 64 ? lane_value(v[0], i) : lane_value(v[R - 1], i - 64);
    }
    __device__ inline void set(int lane, int i, double x) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = lane + 64 * r == i ? x : v[r];
    }
};

// r = sqrt(x) and y = 1 / r for a normal x, each to the last bit but for rare
// ties: the hardware's estimate of 1 / sqrt(x) and one third-order step, the
// root with a residual correction, and a Newton step to that root's reciprocal.
__device__ inline double root_and_reciprocal(double x, double &y) {
    y = __builtin_amdgcn_rsq(x);
    const double h = fma(-x * y, y, 1.0);
    y = fma(y * h, fma(0.375, h, 0.5), y);
    double r = x * y;
    r = fma(0.5 * y, fma(-r, r, x), r);
    y = fma(y, fma(-r, y, 1.0), y);
    return r;
}
// a / r from y = 1 / r, rounded as a division
__device__ inline double quotient(double a, double r, double y) {
    const double q = a * y;
    return fma(fma(-q, r, a), y, q);
}

template <int R>
__device__ void tridiag_ql_first_row(int n, int lane, LaneVec<R> &d, LaneVec<R> &e, LaneVec<R> &z) {
    constexpr double R2_MIN = 1e-280;   // a rotation of smaller squares is one of zeros
#pragma unroll
    for (int r = 0; r < R; ++r) z.v[r] = lane + 64 * r == 0 ? 1.0 : 0.0;
    for (int l = 0; l < n; ++l) {
        int iter = 0;
        while (true) {
            // the first negligible e[mm], l <= mm < n - 1 (else mm = n - 1)
            int mm = n - 1;
#pragma unroll
            for (int r = R - 1; r >= 0; --r) {
                double up = __shfl_down(d.v[r], 1, 64);
                if (r + 1 < R) up = lane == 63 ? lane_value(d.v[R - 1], 0) : up;
                const int i = lane + 64 * r;
                const bool neg = i >= l && i < n - 1 && fabs(e.v[r]) <= DBL_EPSILON * (fabs(d.v[r]) + fabs(up));
                const unsigned long long b = __ballot(neg);
                if (b) mm = 64 * r + __builtin_ctzll(b);
            }
            if (mm == l || ++iter > 64) break;
            const double dl = d.get(l), el = e.get(l);
            double dn = d.get(mm), zn = z.get(mm);   // entries i + 1
            double g = (d.get(l + 1) - dl) / (2.0 * el);
            g = dn - dl + el / (g + copysign(hypot(g, 1.0), g));
            double s = 1.0, c = 1.0, p = 0.0;
            bool early = false;
            int i = mm - 1;
            // rotation i, its entry i in register RD and entry i + 1 in register WR
            auto rotate = [&](auto rd, auto wr) -> bool {
                constexpr int RD = decltype(rd)::value, WR = decltype(wr)::value;
                const int at = i - 64 * RD, to = i + 1 - 64 * WR;
                const double ei = lane_value(e.v[RD], at), di = lane_value(d.v[RD], at), zi = lane_value(z.v[RD], at);
                const double f = s * ei, bb = c * ei, r2 = fma(f, f, g * g);
                if (r2 < R2_MIN) return false;
                double y;
                const double r = root_and_reciprocal(r2, y);
                const bool mine = lane == to;
                e.v[WR] = mine ? r : e.v[WR];
                s = quotient(f, r, y);
                c = quotient(g, r, y);
                g = dn - p;
                const double t = fma(bb, 2.0 * c, s * (di - g));
                d.v[WR] = mine ? fma(s, t, g) : d.v[WR];
                p = s * t;
                g = fma(c, t, -bb);
                z.v[WR] = mine ? fma(c, zn, s * zi) : z.v[WR];
                zn = fma(c, zi, -(s * zn));
                dn = di;
                return true;
            };
            constexpr std::integral_constant<int, 0> r0{};
            constexpr std::integral_constant<int, R - 1> r1{};
            auto walk = [&](auto rd, auto wr, int last) {
                for (; i >= last; --i)
                    if (!rotate(rd, wr)) {
                        early = true;
                        break;
                    }
            };
            if constexpr (R > 1) {
                if (i > 63) walk(r1, r1, l > 64 ? l : 64);
                if (!early && i == 63) walk(r0, r1, l > 63 ? l : 63);
                if (!early) walk(r0, r0, l);
            } else {
                walk(r0, r0, l);
            }
            if (early) {
                d.set(lane, i + 1, dn - p);
                z.set(lane, i + 1, zn);
                e.set(lane, i + 1, 0.0);
                e.set(lane, mm, 0.0);
                continue;
            }
            d.set(lane, l, dn - p);
            z.set(lane, l, zn);
            e.set(lane, l, g);
            e.set(lane, mm, 0.0);
        }
    }
}

// F[k][j-1] = sum_i tau_i^2 |theta_i| for T_j (j capped at steps[k]).
// f of the quadrature: TNSLQ_F_ABS |x| (the negativity), TNSLQ_F_ENTROPY
// -x log2 x (0 for x <= 0), TNSLQ_F_PURITY x^2.
__device__ inline double quad_f(int fn, double x) {
    if (fn == TNSLQ_F_ENTROPY) return x > 0.0 ? -x * log2(x) : 0.0;
    if (fn == TNSLQ_F_PURITY) return x * x;
    return fabs(x);
}

// One wave per (probe, step).  What bounds it is the chain of one problem's
// rotations (about 0.85 m^2 of them, each 20 dependent FP64 operations), not
// the number of problems; with one thread per problem the 32 threads of a
// block also waited for each other's branches.  945 us before, 317 now,
// for 32 probes and 40 steps (280 and 96 for 16 probes and 20 steps).
template <int R>
__device__ inline void quadrature_wave(const double *__restrict__ ak, const double *__restrict__ bk, int jj, int fn,
                                       double *sh) {
    const int lane = threadIdx.x;
    LaneVec<R> d, e, z;
    double big = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = lane + 64 * r;
        d.v[r] = i < jj ? ak[i] : 0.0;
        e.v[r] = i + 1 < jj ? bk[i + 1] : 0.0;
        big = fmax(big, fmax(fabs(d.v[r]), fabs(e.v[r])));
    }
    for (int o = 32; o > 0; o >>= 1) big = fmax(big, __shfl_xor(big, o, 64));
    // scaled by a power of two, so that the squares of a rotation stay normal
    const int x = big > 0.0 && isfinite(big) ? ilogb(big) : 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        d.v[r] = ldexp(d.v[r], -x);
        e.v[r] = ldexp(e.v[r], -x);
    }
    tridiag_ql_first_row<R>(jj, lane, d, e, z);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        sh[lane + 64 * r] = z.v[r] * z.v[r];
        sh[TNSLQ_MAX_STEPS + lane + 64 * r] = quad_f(fn, ldexp(d.v[r], x));
    }
}

__global__ void __launch_bounds__(64) k_quadrature(const double *__restrict__ alpha,
                                                   const double *__restrict__ beta,
                                                   const int *__restrict__ steps, int64_t K, int m, int jlo, int nj,
                                                   int fn, double *__restrict__ F) {
    __shared__ double sh[2 * TNSLQ_MAX_STEPS];   // tau^2, f(theta)
    for (int64_t t = blockIdx.x; t < K * nj; t += gridDim.x) {
        const int64_t k = t % K;
        const int j = jlo + nj - 1 - (int)(t / K);   // the longest chains start first
        int jj = j;
        if (steps && steps[k] < jj) jj = steps[k];
        const double *ak = alpha + k * m, *bk = beta + k * (m + 1);
        if (jj <= 64)
            quadrature_wave<1>(ak, bk, jj, fn, sh);
        else
            quadrature_wave<2>(ak, bk, jj, fn, sh);
        __syncthreads();
        if (threadIdx.x == 0) {
            double f = 0.0;
            for (int i = 0; i < jj; ++i) f = fma(sh[i], sh[TNSLQ_MAX_STEPS + i], f);
            F[k * m + (j - 1)] = f;
        }
        __syncthreads();
    }
}

// G_k = beta_1^2 F_j; mean, SE = sqrt(Var / K) (sample variance), E = log2 mean,
// dE = SE / (mean ln 2).  stats[(j-1)*4 + {0,1,2,3}].  A second block, where
// there is one, takes step j2 (without its G).
__global__ void __launch_bounds__(256) k_stats(const double *__restrict__ beta, const double *__restrict__ F,
                                               int K, int m, int j, int j2, double *__restrict__ G,
                                               double *__restrict__ stats) {
    __shared__ double sh[16];
    if (blockIdx.x == 1) {
        j = j2;
        G = nullptr;
    }
    double s = 0.0;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const double b1 = beta[(int64_t)k * (m + 1)];
        const double g = b1 * b1 * F[(int64_t)k * m + (j - 1)];
        if (G) G[k] = g;
        s += g;
    }
    const double mean = block_sum(s, sh) / K;
    double v = 0.0;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const double b1 = beta[(int64_t)k * (m + 1)];
        const double g = b1 * b1 * F[(int64_t)k * m + (j - 1)];
        v += (g - mean) * (g - mean);
    }
    v = block_sum(v, sh);
    if (threadIdx.x == 0) {
        const double nan = __longlong_as_double(0x7ff8000000000000ll);
        const double se = K > 1 ? sqrt(v / (K - 1) / K) : nan;
        double *o = stats + (int64_t)(j - 1) * 4;
        o[0] = mean;
        o[1] = se;
        o[2] = log2(mean);
        o[3] = K > 1 ? se / (mean * 0.69314718055994530942) : nan;
    }
}

// ---------------------------------------------------------------- fit
// lanczos_estimate of Sec. III: a least-squares fit of F_inf + a r^t to the
// last FIT_WINDOW quadrature values of a probe, leaving out F_1 (the one-node
// rule) (t = 0 at the first point of the window), r in [-FIT_R_MAX, FIT_R_MAX] so that the sign-alternating approach
// of the |x| quadrature is an exponential too.  For fixed r the fit is the
// linear regression of the values on r^t; r is chosen on an even grid of
// FIT_GRID points and refined by golden-section search between the best grid
// point's neighbours.  The fit's own uncertainty of F_inf is sqrt(C_00) of
// C = RSS / (n - 3) (J^T J)^-1, J the model's Jacobian in (F_inf, a, r); an
// exact fit has uncertainty 0, a singular J^T J with RSS > 0 infinity.  To it
// is added in quadrature the model error: the distance from F_inf to the limit
// F_alg of the algebraic law F_j = F_alg + c (-1)^j / j^2 + d / j^2 (j the step
// number) fitted to the same window by linear least squares, the way Gauss
// quadrature of a function with a kink approaches its limit.  A probe whose
// recurrence broke down by step j is exact: F_s, uncertainty 0.
constexpr int FIT_WINDOW = TNSLQ_FIT_WINDOW;
constexpr int FIT_MIN_POINTS = TNSLQ_FIT_MIN_POINTS;
constexpr int FIT_GRID = 397;
constexpr double FIT_R_MAX = 0.99;

// RSS of the regression y_t ~ f + a r^t (t = 0..n-1), with f, a.
__device__ inline double fit_linear(const double *y, int n, double r, double &f, double &a) {
    double x[FIT_WINDOW];
    double p = 1.0, mx = 0.0, my = 0.0;
    for (int t = 0; t < n; ++t) {
        x[t] = p;
        p *= r;
        mx += x[t];
        my += y[t];
    }
    mx /= n;
    my /= n;
    double sxx = 0.0, sxy = 0.0;
    for (int t = 0; t < n; ++t) {
        sxx += (x[t] - mx) * (x[t] - mx);
        sxy += (x[t] - mx) * (y[t] - my);
    }
    a = sxx > 0.0 ? sxy / sxx : 0.0;
    f = my - a * mx;
    double rss = 0.0;
    for (int t = 0; t < n; ++t) {
        const double e = y[t] - f - a * x[t];
        rss += e * e;
    }
    return rss;
}

__device__ inline double fit_grid_r(int i) { return -FIT_R_MAX + (2.0 * FIT_R_MAX) * i / (FIT_GRID - 1); }

// F_alg of the least-squares fit of F_alg + c (-1)^j / j^2 + d / j^2 to the n
// values y of steps j0 .. j0 + n - 1: the two decaying columns are
// orthonormalised (Gram-Schmidt, each projection applied twice) and F_alg is
// the regression of y on the constant column's remainder.
__device__ inline double fit_algebraic(const double *y, int n, int j0) {
    double q[2][FIT_WINDOW], one[FIT_WINDOW], yr[FIT_WINDOW];
    for (int t = 0; t < n; ++t) {
        const double jj = (double)(j0 + t), w = 1.0 / (jj * jj);
        q[0][t] = ((j0 + t) & 1) ? -w : w;
        q[1][t] = w;
        one[t] = 1.0;
        yr[t] = y[t];
    }
    auto dot = [&](const double *u, const double *v) {
        double s = 0.0;
        for (int t = 0; t < n; ++t) s += u[t] * v[t];
        return s;
    };
    auto remove = [&](double *v, const double *u) {
        for (int pass = 0; pass < 2; ++pass) {
            const double c = dot(u, v);
            for (int t = 0; t < n; ++t) v[t] -= c * u[t];
        }
    };
    for (int c = 0; c < 2; ++c) {
        if (c == 1) remove(q[1], q[0]);
        const double nr = sqrt(dot(q[c], q[c]));
        for (int t = 0; t < n; ++t) q[c][t] /= nr;
    }
    for (int c = 0; c < 2; ++c) {
        remove(one, q[c]);
        remove(yr, q[c]);
    }
    return dot(one, yr) / dot(one, one);
}

// Per probe k (one wave each): F_inf and its uncertainty after step
// j >= FIT_MIN_POINTS + 1.  The lanes share the grid; the first grid point of
// least RSS wins (as a scan in order would pick it), and lane 0 refines it.
__global__ void __launch_bounds__(64) k_fit(const double *__restrict__ alpha, const double *__restrict__ beta,
                                            const double *__restrict__ F, int K, int m, int j,
                                            double *__restrict__ finf, double *__restrict__ fsig) {
    const int k = blockIdx.x, lane = threadIdx.x;
    if (k >= K) return;
    const double *ak = alpha + (int64_t)k * m, *bk = beta + (int64_t)k * (m + 1), *Fk = F + (int64_t)k * m;
    const int s = first_break(ak, bk, j);
    if (s > 0) {
        if (lane == 0) {
            finf[k] = Fk[s - 1];
            fsig[k] = 0.0;
        }
        return;
    }
    const int lo = j - FIT_WINDOW > 1 ? j - FIT_WINDOW : 1;   // F_1 is never fitted
    const int n = j - lo;
    double y[FIT_WINDOW];
    for (int t = 0; t < n; ++t) y[t] = Fk[lo + t];
    double f, a, best = INFINITY;
    int ib = FIT_GRID;   // none yet
    for (int i = lane; i < FIT_GRID; i += 64) {
        const double rss = fit_linear(y, n, fit_grid_r(i), f, a);
        if (rss < best) {
            best = rss;
            ib = i;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double ob = __shfl_xor(best, off, 64);
        const int oi = __shfl_xor(ib, off, 64);
        if (ob < best || (ob == best && oi < ib)) {
            best = ob;
            ib = oi;
        }
    }
    if (lane != 0) return;
    if (ib == FIT_GRID) ib = 0;
    double lo_r = fit_grid_r(ib > 0 ? ib - 1 : 0), hi_r = fit_grid_r(ib < FIT_GRID - 1 ? ib + 1 : FIT_GRID - 1);
    const double g = 0.61803398874989484820;   // (sqrt(5) - 1) / 2
    double x1 = hi_r - g * (hi_r - lo_r), x2 = lo_r + g * (hi_r - lo_r);
    double f1 = fit_linear(y, n, x1, f, a), f2 = fit_linear(y, n, x2, f, a);
    for (int it = 0; it < 200 && hi_r - lo_r > 1e-13; ++it) {
        if (f1 <= f2) {
            hi_r = x2;
            x2 = x1;
            f2 = f1;
            x1 = hi_r - g * (hi_r - lo_r);
            f1 = fit_linear(y, n, x1, f, a);
        } else {
            lo_r = x1;
            x1 = x2;
            f1 = f2;
            x2 = lo_r + g * (hi_r - lo_r);
            f2 = fit_linear(y, n, x2, f, a);
        }
    }
    double r = 0.5 * (lo_r + hi_r);
    double rss = fit_linear(y, n, r, f, a);
    if (!(rss <= best)) {
        r = fit_grid_r(ib);
        rss = fit_linear(y, n, r, f, a);
    }
    double sig;
    if (rss == 0.0) {
        sig = 0.0;
    } else {
        // J^T J for the columns 1, r^t, a t r^(t-1)
        double m00 = 0, m01 = 0, m02 = 0, m11 = 0, m12 = 0, m22 = 0;
        double p = 1.0, pm = 1.0;   // r^t, r^(t-1) (taken as 1 at t = 0, where the column is 0)
        for (int t = 0; t < n; ++t) {
            const double c1 = p, c2 = t > 0 ? a * t * pm : 0.0;
            m00 += 1.0;
            m01 += c1;
            m02 += c2;
            m11 += c1 * c1;
            m12 += c1 * c2;
            m22 += c2 * c2;
            pm = p;
            p *= r;
        }
        const double cof00 = m11 * m22 - m12 * m12;
        const double det = m00 * cof00 - m01 * (m01 * m22 - m12 * m02) + m02 * (m01 * m12 - m11 * m02);
        const double c00 = rss / (n - 3) * cof00 / det;
        sig = (det > 0.0 && isfinite(c00) && c00 >= 0.0) ? sqrt(c00) : INFINITY;
    }
    const double dm = f - fit_algebraic(y, n, lo + 1);
    finf[k] = f;
    fsig[k] = isfinite(sig) ? sqrt(sig * sig + dm * dm) : sig;
}

// Block statistics of the fitted estimates: G_n = beta_1^2 F_inf,n;
// out = {mean T, SE (N - 1), eps_L = mean beta_1^2 sigma_n, E = log2 T,
//        dE = sqrt(SE^2 + eps_L^2) / (T ln 2), SE / (T ln 2)}.
__global__ void __launch_bounds__(256) k_fit_stats(const double *__restrict__ beta, const double *__restrict__ finf,
                                                   const double *__restrict__ fsig, int K, int m,
                                                   double *__restrict__ G, double *__restrict__ out) {
    __shared__ double sh[16];
    double s = 0.0, e = 0.0;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const double b1 = beta[(int64_t)k * (m + 1)];
        const double g = b1 * b1 * finf[k];
        if (G) G[k] = g;
        s += g;
        e += b1 * b1 * fsig[k];
    }
    const double mean = block_sum(s, sh) / K;
    const double eps = block_sum(e, sh) / K;
    double v = 0.0;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        const double b1 = beta[(int64_t)k * (m + 1)];
        const double g = b1 * b1 * finf[k];
        v += (g - mean) * (g - mean);
    }
    v = block_sum(v, sh);
    if (threadIdx.x == 0) {
        const double ln2 = 0.69314718055994530942;
        const double se = K > 1 ? sqrt(v / (K - 1) / K) : 0.0;
        out[0] = mean;
        out[1] = se;
        out[2] = eps;
        out[3] = log2(mean);
        out[4] = sqrt(se * se + eps * eps) / (mean * ln2);
        out[5] = K > 1 ? se / (mean * ln2) : __longlong_as_double(0x7ff8000000000000ll);
    }
}

// Surrogate inputs: probe means of dAB alpha_1..n_early in slots 0..7 and of
// dAB beta_2..n_early+1 in slots 8..15 (slots past n_early hold zero), then
// log2 dA, log2 dB, log2 dE.
__global__ void k_features(const double *__restrict__ alpha, const double *__restrict__ beta, int K, int m,
                           int n_early, double dAB, double dA, double dB, double dE, float *__restrict__ feat) {
    const int t = threadIdx.x;
    if (t < 2 * TNSLQ_SURROGATE_MAX_EARLY) {
        const bool is_a = t < TNSLQ_SURROGATE_MAX_EARLY;
        const int i = is_a ? t : t - TNSLQ_SURROGATE_MAX_EARLY;
        double s = 0.0;
        if (i < n_early)
            for (int k = 0; k < K; ++k)
                s += is_a ? alpha[(int64_t)k * m + i] : beta[(int64_t)k * (m + 1) + i + 1];
        feat[t] = (float)(dAB * s / K);
    } else if (t < 2 * TNSLQ_SURROGATE_MAX_EARLY + 3) {
        const int i = t - 2 * TNSLQ_SURROGATE_MAX_EARLY;
        feat[t] = (float)log2(i == 0 ? dA : (i == 1 ? dB : dE));
    }
}

}  // namespace

hipError_t launch_passA(int accfp64, const LzDims &z, const void *part, int S, int64_t split_stride, int k0,
                        int kc, const double2 *q_prev, const double2 *q_cur, double2 *w, const double *alpha,
                        const double *beta, int j, double *dotpart, hipStream_t st, uint64_t *start) {
    dim3 grid(z.nblk, kc), block(256);
    if (accfp64)
        hipLaunchKernelGGL((k_passA<double2>), grid, block, 0, st, (const double2 *)part, S, split_stride, k0,
                           z.n, q_prev, q_cur, w, alpha, beta, z.m, j, z.nblk, dotpart, start);
    else
        hipLaunchKernelGGL((k_passA<float2>), grid, block, 0, st, (const float2 *)part, S, split_stride, k0,
                           z.n, q_prev, q_cur, w, alpha, beta, z.m, j, z.nblk, dotpart, start);
    return hipGetLastError();
}

hipError_t launch_passB(const LzDims &z, const double *dotpart, const double2 *q_cur, double2 *w,
                        double *alpha, const double *beta, int j, double *nrmpart, hipStream_t st, uint64_t *start) {
    dim3 grid(z.nblk, z.K), block(256);
    hipLaunchKernelGGL(k_passB, grid, block, 0, st, dotpart, z.n, q_cur, w, alpha, beta, z.m, j, z.nblk,
                       nrmpart, start);
    return hipGetLastError();
}

hipError_t launch_reorth(const LzDims &z, const double *dotpart, const double2 *Q, int64_t slot, double2 *w,
                         double *hpart, double2 *h, double *alpha, const double *beta, int j, double *nrmpart,
                         hipStream_t st, uint64_t *start) {
    const int bt = reorth_chunk(z.n, z.K);
    const int64_t chunks = reorth_chunks(z.n, z.K);
    if (chunks > 0x7fffffff) return hipErrorInvalidConfiguration;
    const int nc = (int)chunks;
    const bool fold = nc <= REORTH_FOLD;
    double2 *p0 = (double2 *)hpart, *p1 = fold ? p0 + (size_t)z.K * j * nc : p0;
    const dim3 grid(nc, z.K), block(bt), rgrid((j + 3) / 4, z.K);
    hipLaunchKernelGGL(k_passB_dots, grid, block, 0, st, dotpart, z.nblk, z.n, Q, slot, w, alpha, beta, z.m, j, nc, p0,
                       start);
    if (!fold) hipLaunchKernelGGL(k_reorth_reduce, rgrid, dim3(256), 0, st, (const double2 *)p0, j, nc, h);
    hipLaunchKernelGGL(k_reorth_update_dots, grid, block, 0, st, Q, j, slot, z.n, (const double2 *)h,
                       (const double2 *)p0, w, nc, p1);
    if (!fold) hipLaunchKernelGGL(k_reorth_reduce, rgrid, dim3(256), 0, st, (const double2 *)p1, j, nc, h);
    hipLaunchKernelGGL(k_reorth_update, dim3(z.nblk, z.K), dim3(256), 0, st, Q, j, slot, z.n, (const double2 *)h,
                       (const double2 *)p1, nc, w, z.nblk, nrmpart);
    return hipGetLastError();
}

hipError_t launch_passC(int prec, const LzDims &z, const double *nrmpart, const double2 *w, double2 *q_next,
                        void *Xt, int64_t xt_nst, const double *alpha, double *beta, int j, hipStream_t st) {
    // whole tiles per block where the pass transposes into Xt
    dim3 grid((unsigned)(Xt ? std::min<int64_t>(xt_tiles(z.dA, z.dB), 1024) : z.nblk), z.K), block(256);
#define TNSLQ_PC(P)                                                                                         \
    hipLaunchKernelGGL((k_passC<P>), grid, block, 0, st, nrmpart, z.n, z.dA, z.dB, w, q_next, Xt, xt_nst, \
                       alpha, beta, z.m, j, z.nblk)
    switch (prec) {
        case TNSLQ_FP64: TNSLQ_PC(TNSLQ_FP64); break;
        case TNSLQ_FP32: TNSLQ_PC(TNSLQ_FP32); break;
        case TNSLQ_BF16X3: TNSLQ_PC(TNSLQ_BF16X3); break;
        default: TNSLQ_PC(TNSLQ_BF16X6); break;
    }
#undef TNSLQ_PC
    return hipGetLastError();
}

hipError_t launch_steps(const double *alpha, const double *beta, int K, int m, int jdone, int *steps,
                        hipStream_t st, uint64_t *start) {
    hipLaunchKernelGGL(k_steps, dim3(K), dim3(64), 0, st, alpha, beta, m, jdone, steps, start);
    return hipGetLastError();
}

hipError_t launch_quadrature(const double *alpha, const double *beta, const int *steps, int K, int m, int jlo,
                             int jhi, int fn, double *F, hipStream_t st) {
    const int nj = jhi - jlo + 1;
    const int64_t nt = (int64_t)K * nj;
    hipLaunchKernelGGL(k_quadrature, dim3((unsigned)(nt < (1 << 20) ? nt : (1 << 20))), dim3(64), 0, st, alpha, beta,
                       steps, (int64_t)K, m, jlo, nj, fn, F);
    return hipGetLastError();
}

hipError_t launch_stats(const double *beta, const double *F, int K, int m, int j, int j2, double *G, double *stats,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_stats, dim3(j2 > 0 ? 2 : 1), dim3(256), 0, st, beta, F, K, m, j, j2, G, stats);
    return hipGetLastError();
}

hipError_t launch_fit(const double *alpha, const double *beta, const double *F, int K, int m, int j, double *finf,
                      double *fsig, double *G, double *out, hipStream_t st) {
    if (j < FIT_MIN_POINTS + 1 || j > m) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fit, dim3(K), dim3(64), 0, st, alpha, beta, F, K, m, j, finf, fsig);
    hipLaunchKernelGGL(k_fit_stats, dim3(1), dim3(256), 0, st, beta, (const double *)finf, (const double *)fsig, K, m,
                       G, out);
    return hipGetLastError();
}

hipError_t launch_features(const double *alpha, const double *beta, int K, int m, int n_early, double dAB,
                           double dA, double dB, double dE, float *feat, hipStream_t st) {
    hipLaunchKernelGGL(k_features, dim3(1), dim3(64), 0, st, alpha, beta, K, m, n_early, dAB, dA, dB, dE, feat);
    return hipGetLastError();
}

}  // namespace tnslq
