// Whole Lanczos steps of a small explicit operator in one launch (FP64,
// n = d_A d_B <= 128).  Such a step is a few microseconds of work; as four to
// six kernels it was their launches and the latencies at their ends.  Here a
// block takes 16 probes, the columns of one matrix-instruction tile, through
// all the steps asked for, and probes share nothing else:
//   product     one wave per 16 rows of rho^{T_B}: fragments of rho from its
//               bricks (from the caches, one brick ahead), of the vectors from
//               LDS, outputs to LDS;
//   recurrence  one wave per probe, the vector and its predecessor in
//               registers (one or two elements per lane), every sum a wave's.
// Two barriers a step.  The matrix instructions bound the product, n^2 cycles
// with four SIMDs: 1.7 us at n = 64 and 6.8 us at 128, where the general step's
// five launches (and their gaps) are level with it; beyond, more CUs are worth
// more than fewer launches.  Products and sums are those of the general
// kernels, in their order, so that the results are the same bit for bit.
// n = 64, 16 probes, 20 steps: 400 us in 80 launches to 82 us in one.
#include "breakdown.h"
#include "gemm_tiles.h"
#include "tnslq_internal.h"

namespace tnslq {
namespace {

constexpr int SM_PROBES = 16;

// XN: elements per lane, n <= 64 XN
template <int XN>
__global__ void __launch_bounds__(64 * SM_PROBES) k_small_steps(SmallSteps g) {
#pragma clang fp contract(off)   // roundings as written: those of the general kernels
    constexpr int N = 64 * XN;
    constexpr int BRICKB = MP<TNSLQ_FP64>::NPL * TILEB;
    __shared__ __attribute__((aligned(16))) double xs[2][SM_PROBES][N + 2];   // Re, Im of the vectors
    __shared__ double2 ys[SM_PROBES][N + 1];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 15, fk = lane >> 4;
    const int n = g.n, k = blockIdx.x * SM_PROBES + wid;
    const bool have = k < g.K;
    const int64_t at = (int64_t)k * n + lane;   // this lane's elements: at + 64 x
    double *ak = g.alpha + (int64_t)k * g.m, *bk = g.beta + (int64_t)k * (g.m + 1);
    auto slot_of = [&](int j) { return (g.reorth ? j : j % 3) * g.slot; };
    double2 q[XN], qp[XN];
    bool in[XN];
    double amax = 0.0, bmax = 0.0, bj = 0.0;
    bool live = false;
#pragma unroll
    for (int x = 0; x < XN; ++x) {
        in[x] = have && lane + 64 * x < n;
        q[x] = in[x] ? g.Q[slot_of(g.j0 - 1) + at + 64 * x] : make_double2(0.0, 0.0);
        qp[x] = in[x] && g.j0 > 1 ? g.Q[slot_of(g.j0 - 2) + at + 64 * x] : make_double2(0.0, 0.0);
    }
    if (have) {
        live = first_break(ak, bk, g.j0 - 1, amax, bmax) == 0;
        if (g.j0 > 1) bj = bk[g.j0 - 1];
    }
    // a sum over the vector from the lanes' terms: 64 elements at a time
    auto total = [&](const double (&t)[XN]) {
        double s = 0.0;
#pragma unroll
        for (int x = 0; x < XN; ++x) s += wave_tree_total(t[x]);
        return s;
    };
    for (int j = g.j0; j <= g.j1; ++j) {
#pragma unroll
        for (int x = 0; x < XN; ++x) {
            xs[0][wid][lane + 64 * x] = q[x].x;
            xs[1][wid][lane + 64 * x] = q[x].y;
        }
        uint64_t *t = g.stamps + (j - 1) * g.step_stamps;
        stamp(t);
        __syncthreads();
        if (16 * wid < n) {
            const char *ga = (const char *)g.rho + loff(16 * wid + frow, fk);
            auto load = [&](int st, uint4 (&fa)[1][2]) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < 2; ++p) fa[0][p] = *(const uint4 *)(ga + st * BRICKB + p * TILEB);
            };
            f64x4 yr = {0, 0, 0, 0}, yi = {0, 0, 0, 0};
            uint4 fa[2][1][2];
            load(0, fa[0]);
            // the general product's splits, one after the other
            for (int s = 0, st = 0; s < g.S; ++s) {
                const int send = g.nst * (s + 1) / g.S;
                f64x4 accr[1][1] = {{{0, 0, 0, 0}}}, acci[1][1] = {{{0, 0, 0, 0}}};
                for (; st < send; ++st) {
                    load(st + 1 < g.nst ? st + 1 : st, fa[1]);
                    uint4 fb[1][2];
#pragma unroll
                    for (int p = 0; p < 2; ++p) fb[0][p] = *(const uint4 *)&xs[p][frow][8 * st + 2 * fk];
                    stage_mfma<TNSLQ_FP64, 1, 1>(fa[0], fb, accr, acci);
                    fa[0][0][0] = fa[1][0][0];
                    fa[0][0][1] = fa[1][0][1];
                }
                yr += accr[0][0];
                yi += acci[0][0];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) ys[frow][16 * wid + 4 * r + fk] = make_double2(yr[r], yi[r]);
        }
        __syncthreads();
        stamp(t + g.merge_stamp);
        stamp(t + g.lanczos_stamp);
        if (!have) continue;
        // w = Y - beta_j q_{j-1}, alpha_j = Re<q_j, w>
        double2 v[XN];
        double acc[XN];
#pragma unroll
        for (int x = 0; x < XN; ++x) {
            const double2 y = ys[wid][lane + 64 * x];
            double re = y.x, im = y.y;
            if (j > 1) {
                re = fma(-bj, qp[x].x, re);
                im = fma(-bj, qp[x].y, im);
            }
            if (!live || !in[x]) re = im = 0.0;
            v[x] = make_double2(re, im);
            acc[x] = fma(q[x].x, re, q[x].y * im);
        }
        double a = total(acc);
        if (!live) a = 0.0;
#pragma unroll
        for (int x = 0; x < XN; ++x) {
            v[x].x = fma(-a, q[x].x, v[x].x);
            v[x].y = fma(-a, q[x].y, v[x].y);
        }
        // Gram-Schmidt twice against q_1 .. q_j, four at a time (zeros past
        // q_j); lane i keeps h_i
        constexpr int U = 4;
        auto stored = [&](int i, int x) {
            return in[x] && i < j ? g.Q[i * g.slot + at + 64 * x] : make_double2(0.0, 0.0);
        };
        for (int pass = 0; pass < 2 * g.reorth; ++pass) {
            double hr = 0.0, hi = 0.0;
            for (int i0 = 0; i0 < j; i0 += U) {
                double2 c[U][XN];
                double sr[U], si[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    sr[u] = si[u] = 0.0;
#pragma unroll
                    for (int x = 0; x < XN; ++x) c[u][x] = stored(i0 + u, x);
                }
#pragma unroll
                for (int x = 0; x < XN; ++x)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        // conj(c) * v
                        sr[u] += wave_total(fma(c[u][x].y, v[x].y, c[u][x].x * v[x].x));
                        si[u] += wave_total(fma(c[u][x].x, v[x].y, -(c[u][x].y * v[x].x)));
                    }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (lane == i0 + u) {
                        hr = sr[u];
                        hi = si[u];
                    }
            }
            for (int i0 = 0; i0 < j; i0 += U)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double cx = lane_value(hr, i0 + u), cy = lane_value(hi, i0 + u);
#pragma unroll
                    for (int x = 0; x < XN; ++x) {
                        const double2 c = stored(i0 + u, x);
                        v[x].x -= fma(cx, c.x, -(cy * c.y));
                        v[x].y -= fma(cx, c.y, cy * c.x);
                    }
                }
        }
#pragma unroll
        for (int x = 0; x < XN; ++x)
            acc[x] = g.reorth ? fma(v[x].y, v[x].y, v[x].x * v[x].x) : fma(v[x].x, v[x].x, v[x].y * v[x].y);
        double b = sqrt(total(acc));
        if (!live) b = 0.0;
        amax = fmax(amax, fabs(a));
        if (j >= 2) bmax = fmax(bmax, bj);
        live = live && !(b <= BREAKDOWN_TOL * (amax + bmax));
#pragma unroll
        for (int x = 0; x < XN; ++x) {
            qp[x] = q[x];
            q[x] = live ? make_double2(v[x].x / b, v[x].y / b) : make_double2(0.0, 0.0);
            if (in[x]) g.Q[slot_of(j) + at + 64 * x] = q[x];
        }
        bj = b;
        if (lane == 0) {
            ak[j - 1] = a;
            bk[j] = b;
        }
    }
}

}  // namespace

hipError_t launch_small_steps(const SmallSteps &g, hipStream_t st) {
    if (!small_steps_supported(g.n, g.K, g.m, g.reorth) || g.nst != brick_stages(TNSLQ_FP64, g.n) || g.j0 < 1 || g.j1 > g.m)
        return hipErrorInvalidValue;
    const dim3 grid((unsigned)((g.K + SM_PROBES - 1) / SM_PROBES)), block(64 * SM_PROBES);
    if (g.n <= 64)
        hipLaunchKernelGGL(k_small_steps<1>, grid, block, 0, st, g);
    else
        hipLaunchKernelGGL(k_small_steps<2>, grid, block, 0, st, g);
    return hipGetLastError();
}

}  // namespace tnslq
