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
// kernels, in their order, so that the results are the same bit for bit up to 64
// probes or n = 32; more probes on a larger n take three real products per complex
// one there (gemm_mfma.hip) and four here.
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

// Everything after the contraction in one step of short vectors, one block of 16
// waves per probe: passA, passB or the reorthogonalisation, and passC.  As
// three to five kernels, launches and the latencies of small blocks were most
// of it.  A lane holds one element of its wave's unit: 64 elements of a 256-thread
// block of the general passes, at most 16 units (blocks times waves per block; the
// blocks depend on n and on the number of probes: up to 256 probes n <= 768, 896 and
// 1024, at 512 every n up to 1024; two units per wave lost: 14 KB of code that runs once, 33 us
// where the general kernels take 31 at n = 864).  w goes through LDS for the dot
// products, (vector, chunk) pairs of the general kernels dealt to the waves.
// Sums keep the general kernels' order and roundings: the results are the same
// bit for bit.  Reorthogonalisation reads the probe's vectors three times through
// one CU, so that j n is bounded, by 16384 elements (3 x 256 KiB).  Estimates on
// qubits, 20 steps: n = 256, 8 probes 982 to 698 us reorthogonalised and 675 to
// 512 not; n = 512, 16 probes 989 to 775; with the bound at 32768, 30 steps of 32
// probes at n = 1024 took 1880 us instead of 1843.
constexpr int SR_WAVES = STEP_REST_UNITS;
constexpr int STEP_REST_MAX_PAIRS = 1024;    // (vector, chunk) pairs of the dot products

template <typename AccT, int PREC>
__global__ void __launch_bounds__(64 * SR_WAVES) k_step_rest(StepRest g) {
#pragma clang fp contract(off)   // roundings as written: those of the general kernels
    __shared__ double2 ws[STEP_REST_MAX_N];
    __shared__ double2 hs[TNSLQ_MAX_STEPS + 1];
    __shared__ double2 hp[STEP_REST_MAX_PAIRS];
    __shared__ double part[2][SR_WAVES];
    stamp(g.merge_stamp);
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = g.n, k = blockIdx.x, j = g.j;
    const double *ak = g.alpha + (int64_t)k * g.m;
    const double *bk = g.beta + (int64_t)k * (g.m + 1);
    const int64_t base = (int64_t)k * n;
    // units: blocks of `chunk` elements, wpb waves each
    const int chunk = (n + g.nblk - 1) / g.nblk, wpb = (chunk + 63) / 64;
    const int e = wid / wpb * chunk + 64 * (wid % wpb) + lane;
    const bool in = wid / wpb < g.nblk && 64 * (wid % wpb) + lane < chunk && e < n;
    // loads first, then the breakdown test while they are in flight
    double2 q = make_double2(0.0, 0.0), qp = q, v = q;
    if (in) {
        q = g.q_cur[base + e];
        if (j > 1) qp = g.q_prev[base + e];
        for (int s = 0; s < g.S; ++s) {
            const AccT p = ((const AccT *)g.part)[s * g.split + base + e];
            v.x += (double)p.x;
            v.y += (double)p.y;
        }
    }
    const double bj = j > 1 ? bk[j - 1] : 0.0;
    double amax, bmax;
    const bool live = first_break(ak, bk, j - 1, amax, bmax) == 0;
    // the vector's sum from the lanes' terms: units, blocks, then the blocks'
    // tree; buffer p of the two alternates between the sums of a step
    auto total = [&](double t, int p) {
        t = wave_tree_total(in ? t : 0.0);
        if (lane == 0) part[p][wid] = t;
        __syncthreads();
        double s = 0.0;
        if (lane < g.nblk)
            for (int c = 0; c < wpb; ++c) s += part[p][lane * wpb + c];
        return 0.0 + wave_tree_total(s);
    };
    // w = Y - beta_j q_{j-1}, alpha_j = Re<q_j, w>, w -= alpha_j q_j
    if (j > 1) {
        v.x = fma(-bj, qp.x, v.x);
        v.y = fma(-bj, qp.y, v.y);
    }
    if (!live) v = make_double2(0.0, 0.0);
    double a = total(fma(q.x, v.x, q.y * v.y), 0);
    if (!live) a = 0.0;
    stamp(g.lanczos_stamp);
    v.x = fma(-a, q.x, v.x);
    v.y = fma(-a, q.y, v.y);
    // Gram-Schmidt twice against q_1 .. q_j
    for (int pass = 0; pass < 2 * g.reorth; ++pass) {
        if (in) ws[e] = v;
        __syncthreads();
        const int nc = (n + g.rchunk - 1) / g.rchunk, items = j * nc;
        constexpr int U = 4;   // (vector, chunk) pairs in flight per wave
        for (int t0 = wid; t0 < items; t0 += SR_WAVES * U) {
            double re[U], im[U];
#pragma unroll
            for (int u = 0; u < U; ++u) re[u] = im[u] = 0.0;
            for (int x = lane; x < g.rchunk; x += 64) {
                double2 c[U], w[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int it = t0 + SR_WAVES * u, at = (it % nc) * g.rchunk + x;
                    const bool ok = it < items && at < n;
                    c[u] = ok ? g.Q[(it / nc) * g.slot + base + at] : make_double2(0.0, 0.0);
                    w[u] = ok ? ws[at] : make_double2(0.0, 0.0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {   // conj(c) * w
                    re[u] += fma(c[u].y, w[u].y, c[u].x * w[u].x);
                    im[u] += fma(c[u].x, w[u].y, -(c[u].y * w[u].x));
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double sr = wave_total(re[u]), si = wave_total(im[u]);
                if (lane == 0 && t0 + SR_WAVES * u < items) hp[t0 + SR_WAVES * u] = make_double2(sr, si);
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < j) {
            double2 h = make_double2(0.0, 0.0);
            for (int c = 0; c < nc; ++c) {
                const double2 p = hp[threadIdx.x * nc + c];
                h.x += p.x;
                h.y += p.y;
            }
            hs[threadIdx.x] = h;
        }
        __syncthreads();
        const double2 *qe = g.Q + base + e;
        if (in)
#pragma unroll 8
            for (int i = 0; i < j; ++i) {
                const double2 c = qe[i * g.slot], h = hs[i];
                v.x -= fma(h.x, c.x, -(h.y * c.y));
                v.y -= fma(h.x, c.y, h.y * c.x);
            }
    }
    // beta_{j+1} = ||w||, q_{j+1} = w / beta_{j+1}, 0 after a breakdown
    double b = sqrt(total(g.reorth ? fma(v.y, v.y, v.x * v.x) : fma(v.x, v.x, v.y * v.y), 1));
    if (!live) b = 0.0;
    amax = fmax(amax, fabs(a));
    if (j >= 2) bmax = fmax(bmax, bj);
    const bool cont = live && !(b <= BREAKDOWN_TOL * (amax + bmax));
    if (in) {
        const double2 r = cont ? make_double2(v.x / b, v.y / b) : make_double2(0.0, 0.0);
        g.q_next[base + e] = r;
        if (g.Xt)
            store_planes<PREC>(g.Xt, brick_ps(PREC),
                               brick_index(PREC, g.xt_nst, (int64_t)k * g.dB + e % g.dB, e / g.dB), r.x, r.y);
    }
    if (threadIdx.x == 0) {
        g.alpha[(int64_t)k * g.m + j - 1] = a;
        g.beta[(int64_t)k * (g.m + 1) + j] = b;
    }
}

}  // namespace

hipError_t launch_step_rest(int accfp64, int prec, const StepRest &g, int K, hipStream_t st) {
    if (!step_rest_supported(g.n, K, g.j, g.reorth, g.nblk) || g.dB < 1 ||
        (g.reorth && (g.rchunk < 64 || (g.n + g.rchunk - 1) / g.rchunk * g.j > STEP_REST_MAX_PAIRS)))
        return hipErrorInvalidValue;
    const dim3 grid(K), block(64 * SR_WAVES);
#define TNSLQ_SR(T, P) hipLaunchKernelGGL((k_step_rest<T, P>), grid, block, 0, st, g)
    if (accfp64)
        TNSLQ_SR(double2, TNSLQ_FP64);
    else if (prec == TNSLQ_FP32)
        TNSLQ_SR(float2, TNSLQ_FP32);
    else if (prec == TNSLQ_BF16X3)
        TNSLQ_SR(float2, TNSLQ_BF16X3);
    else
        TNSLQ_SR(float2, TNSLQ_BF16X6);
#undef TNSLQ_SR
    return hipGetLastError();
}

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
