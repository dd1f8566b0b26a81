// Complex "NT" contraction C = A * B^T over brick operands with few columns
// (N <= 64, FP32 and FP64) or, in FP64, few terms: the explicit operator on a block of
// probes, or few vectors on a small B.  A 128-column tile would be half to
// seven eighths padding, and such a product is bound by reading A once: a wave
// takes one tile of 16 rows against all NTC tiles of 16 columns and loads its
// fragments straight from the bricks into registers (16 rows of a plane are
// 1 KiB of consecutive memory), one brick ahead, with no LDS and no barrier.
// B's bricks (N rows) stay in the caches: the 8 waves of a block of 128 rows
// and one split read the same ones.  The reduction is split in S runs that
// need not be equal, so that any S gives the chip enough waves.  The FP32 sums
// restart every 64 terms and are added in FP64.  n = 4096, 32 columns, FP32:
// 159 to 42 us (the operator's 128 MB once); n = 864, 8 columns, FP64: 104
// to 7 us; n = 64, 16 columns, FP64: 34 to 4 us.
#include "gemm_tiles.h"

namespace tnslq {
namespace {

constexpr int THIN_WAVES = 4;

template <int PREC, int NTC>
__global__ void __launch_bounds__(64 * THIN_WAVES) k_thin_product(GemmDesc g) {
    stamp(g.start);
    using Acc = typename MP<PREC>::acc;
    constexpr int NPL = MP<PREC>::NPL, BRICKB = NPL * TILEB;
    constexpr int FLUSH = PREC == TNSLQ_FP32 ? 4 : 1 << 30;   // bricks per restart (64 terms)
    const int lane = threadIdx.x & 63, frow = lane & 15, fk = lane >> 4;
    // waves: rows of a brick block fastest, then the split, then the block
    const int64_t w = (int64_t)blockIdx.x * THIN_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t rb = (w >> 3) / g.S;
    const int s = (int)((w >> 3) % g.S), r8 = (int)(w & 7);
    const int64_t i0 = rb * BM + 16 * r8;
    if (i0 >= g.M) return;
    const int64_t sbeg = g.nst * s / g.S, send = g.nst * (s + 1) / g.S;
    const char *ga = (const char *)g.A + (size_t)rb * brick_block_bytes(PREC, g.nst) + loff(16 * r8 + frow, fk);
    // columns in groups of 64 (half a row block of B) along the grid's y
    const int64_t cg = blockIdx.y;
    const char *gb = (const char *)g.B + (size_t)(cg >> 1) * brick_block_bytes(PREC, g.nst) + (cg & 1) * (TILEB / 2);
    int ob[NTC];
#pragma unroll
    for (int c = 0; c < NTC; ++c) ob[c] = loff(16 * c + frow, fk);
    auto load = [&](int64_t st, uint4 (&fa)[1][NPL], uint4 (&fb)[NTC][NPL]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NPL; ++p) fa[0][p] = *(const uint4 *)(ga + st * BRICKB + p * TILEB);
#pragma unroll
        for (int c = 0; c < NTC; ++c)
#pragma unroll
            for (int p = 0; p < NPL; ++p) fb[c][p] = *(const uint4 *)(gb + st * BRICKB + p * TILEB + ob[c]);
    };
    Acc accr[1][NTC], acci[1][NTC];
    f64x4 outr[NTC], outi[NTC];
#pragma unroll
    for (int c = 0; c < NTC; ++c) {
        accr[0][c] = acci[0][c] = Acc{0, 0, 0, 0};
        outr[c] = outi[c] = f64x4{0, 0, 0, 0};
    }
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NTC; ++c) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                outr[c][r] += (double)accr[0][c][r];
                outi[c][r] += (double)acci[0][c][r];
            }
            accr[0][c] = acci[0][c] = Acc{0, 0, 0, 0};
        }
    };
    if (sbeg < send) {
        uint4 fa[2][1][NPL], fb[2][NTC][NPL];
        load(sbeg, fa[0], fb[0]);
        int cnt = 0;
        for (int64_t st = sbeg; st < send; st += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (st + h >= send) break;
                load(st + h + 1 < send ? st + h + 1 : send - 1, fa[h ^ 1], fb[h ^ 1]);
                stage_mfma<PREC, 1, NTC>(fa[h], fb[h], accr, acci);
                if (PREC == TNSLQ_FP32 && ++cnt == FLUSH) {
                    flush();
                    cnt = 0;
                }
            }
        }
    }
    if constexpr (PREC == TNSLQ_FP32) {
        flush();
#pragma unroll
        for (int c = 0; c < NTC; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                accr[0][c][r] = (float)outr[c][r];
                acci[0][c][r] = (float)outi[c][r];
            }
    }
    store_tiles<PREC, 1, NTC>(g, s, i0, 64 * cg, lane, accr, acci);
}

template <int PREC>
hipError_t launch_thin(const GemmDesc &g, hipStream_t st) {
    const int64_t waves = (g.M + BM - 1) / BM * 8 * g.S;
    const int64_t nblocks = (waves + THIN_WAVES - 1) / THIN_WAVES;
    if (nblocks < 1 || nblocks > 0xffffff) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)nblocks, (unsigned)((g.N + 63) / 64)), block(64 * THIN_WAVES);
    switch (g.N <= 48 ? (g.N + 15) / 16 : 4) {
        case 1: hipLaunchKernelGGL((k_thin_product<PREC, 1>), grid, block, 0, st, g); break;
        case 2: hipLaunchKernelGGL((k_thin_product<PREC, 2>), grid, block, 0, st, g); break;
        case 3: hipLaunchKernelGGL((k_thin_product<PREC, 3>), grid, block, 0, st, g); break;
        default: hipLaunchKernelGGL((k_thin_product<PREC, 4>), grid, block, 0, st, g); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_thin(int prec, const GemmDesc &g, hipStream_t st) {
    return prec == TNSLQ_FP64 ? launch_thin<TNSLQ_FP64>(g, st) : launch_thin<TNSLQ_FP32>(g, st);
}

}  // namespace tnslq
