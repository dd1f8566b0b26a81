// Complex "NT" contraction C = A * B^T over brick operands with few columns
// (N <= 64, FP32 and FP64) or, in FP64, few terms: the explicit operator on a block of
// probes, or few vectors on a small B.  A 128-column tile would be half to
// seven eighths padding, and such a product is bound by reading A once: a wave
// takes one tile of 16 rows against all NTC tiles of 16 columns and loads its
// fragments straight from the bricks into registers (16 rows of a plane are
// 1 KiB of consecutive memory), one step ahead, with no LDS and no barrier (four
// bricks ahead made no difference).  B's bricks (N rows) stay in the caches: the
// 8 waves of a block of 128 rows and one split read the same ones.  The
// reduction is split in S runs that need not be equal, so that any S gives the
// chip enough waves.  n = 4096, 32 columns, FP32: 159 to 35 us (the operator's
// 128 MB once are 27); n = 864, 8 columns, FP64: 104 to 7 us; n = 64, 16 columns,
// FP64: 34 to 4 us.
#include "gemm_tiles.h"

namespace tnslq {
namespace {

constexpr int THIN_WAVES = 4;

// FP64
template <int NTC>
__global__ void __launch_bounds__(64 * THIN_WAVES) k_thin_product(GemmDesc g) {
    stamp(g.start);
    constexpr int PREC = TNSLQ_FP64, NPL = MP<PREC>::NPL, BRICKB = NPL * TILEB;
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
    f64x4 accr[1][NTC], acci[1][NTC];
#pragma unroll
    for (int c = 0; c < NTC; ++c) accr[0][c] = acci[0][c] = f64x4{0, 0, 0, 0};
    if (sbeg < send) {
        uint4 fa[2][1][NPL], fb[2][NTC][NPL];
        load(sbeg, fa[0], fb[0]);
        for (int64_t st = sbeg; st < send; st += 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (st + h >= send) break;
                load(st + h + 1 < send ? st + h + 1 : send - 1, fa[h ^ 1], fb[h ^ 1]);
                stage_mfma<PREC, 1, NTC>(fa[h], fb[h], accr, acci);
            }
        }
    }
    store_tiles<PREC, 1, NTC>(g, s, i0, 64 * cg, lane, accr, acci);
}

// FP32, on the BF16 matrix cores: each value is the exact sum of three BF16
// pieces, split from the fragments in registers, and a product of two values the
// six products of pieces (p, q) with p + q < 3.  The FP32 unit took 29 us of n =
// 4096's 42 for 32 columns; 24 BF16 instructions per 32 terms are a third less
// and leave the split to the vector units: 35 us, and 20 steps of 64 columns 2.50
// to 2.08 ms.  A step is two bricks: lane (l % 16, l / 16) holds unit l / 16 of
// both as the 8 terms of its BF16 fragment, of A and of B alike.  The products of
// leading pieces and the small ones have accumulators of their own; both restart
// every 128 terms and are added in FP64: a block matvec is off by 0.8e-7 to
// 1.3e-7 of its result, where the FP32 unit with sums restarted every 64 terms
// had 2.0e-7 to 2.9e-7.  GemmDesc::chunk restarts them sooner; two products add to
// each here, so its terms are half as many steps.  Values that the pieces do not
// reach, and results that are not finite, go to that unit (gemm_tiles.h).
constexpr int THIN_FLUSH = 4;   // steps of 32 terms per restart

template <int NTC>
__global__ void __launch_bounds__(64 * THIN_WAVES, 5 - NTC) k_thin_fp32(GemmDesc g) {
    stamp(g.start);
    constexpr int BRICKB = 2 * TILEB;
    const int lane = threadIdx.x & 63, frow = lane & 15, fk = lane >> 4;
    const int64_t w = (int64_t)blockIdx.x * THIN_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t rb = (w >> 3) / g.S;
    const int s = (int)((w >> 3) % g.S), r8 = (int)(w & 7);
    const int64_t i0 = rb * BM + 16 * r8;
    if (i0 >= g.M) return;
    const int64_t sbeg = g.nst * s / g.S, send = g.nst * (s + 1) / g.S;
    const char *ga = (const char *)g.A + (size_t)rb * brick_block_bytes(TNSLQ_FP32, g.nst) + loff(16 * r8 + frow, fk);
    const char *gb = (const char *)g.B;
    // (rows 16 apart have their units in the same order)
    const int ob = loff(frow, fk);
    constexpr int OC = 16 * ROWB;   // from a column tile's rows to the next one's
    // a step's fragments: [plane][brick]; a last odd brick's second half is zeros
    auto load = [&](int64_t st, float4 (&fa)[2][2], float4 (&fb)[NTC][2][2]) __attribute__((always_inline)) {
        const int64_t s1 = st + 1 < send ? st + 1 : st;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            fa[p][0] = *(const float4 *)(ga + st * BRICKB + p * TILEB);
            fa[p][1] = *(const float4 *)(ga + s1 * BRICKB + p * TILEB);
#pragma unroll
            for (int c = 0; c < NTC; ++c) {
                fb[c][p][0] = *(const float4 *)(gb + st * BRICKB + p * TILEB + ob + c * OC);
                fb[c][p][1] = *(const float4 *)(gb + s1 * BRICKB + p * TILEB + ob + c * OC);
            }
        }
    };
    auto split = [&](const float4 (&x)[2], uint4 (&h)[3]) __attribute__((always_inline)) {
        typedef __attribute__((ext_vector_type(2))) float f32x2;
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        uint32_t o[3][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float4 v = x[k >> 1];
            float a = k & 1 ? v.z : v.x, b = k & 1 ? v.w : v.y;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                o[p][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
                a -= __uint_as_float(o[p][k] << 16);
                b -= __uint_as_float(o[p][k] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) h[p] = make_uint4(o[p][0], o[p][1], o[p][2], o[p][3]);
    };
    // [Re, Im][leading, small]
    f32x4 acc[2][2][NTC];
    f64x4 out[2][NTC];
#pragma unroll
    for (int c = 0; c < NTC; ++c)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            acc[x][0][c] = acc[x][1][c] = f32x4{0, 0, 0, 0};
            out[x][c] = f64x4{0, 0, 0, 0};
        }
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NTC; ++c)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
#pragma unroll
                for (int r = 0; r < 4; ++r) out[x][c][r] += (double)acc[x][0][c][r] + (double)acc[x][1][c][r];
                acc[x][0][c] = acc[x][1][c] = f32x4{0, 0, 0, 0};
            }
    };
    float4 fa[2][2], fb[NTC][2][2];
    uint32_t bitsA = 0, bitsB[NTC];   // of the leading pieces (gemm_tiles.h)
#pragma unroll
    for (int c = 0; c < NTC; ++c) bitsB[c] = 0;
    if (sbeg < send) load(sbeg, fa, fb);
    const int every = g.chunk ? (g.chunk + 1) / 2 : THIN_FLUSH;
    int left = every;   // (counted up, two column tiles spilled 40 registers: 20 qubits 4.6 ms for 4.07)
    for (int64_t st = sbeg; st < send; st += 2) {
        if (st + 1 >= send) {
#pragma unroll
            for (int p = 0; p < 2; ++p) fa[p][1] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        uint4 ha[2][3], na[3], hb[NTC][2][3];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            split(fa[p], ha[p]);
            bitsA |= or_bits(ha[p][0]);
#pragma unroll
            for (int c = 0; c < NTC; ++c) {
                split(fb[c][p], hb[c][p]);
                bitsB[c] |= or_bits(hb[c][p][0]);
            }
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) na[p] = neg_bf16x8(ha[1][p]);
        load(st + 2 < send ? st + 2 : send - 1, fa, fb);
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) {
            // (0,0), (0,1), (1,0), (1,1), (0,2), (2,0)
            const int p = pq == 2 || pq == 3 ? 1 : (pq == 5 ? 2 : 0);
            const int q = pq == 1 || pq == 3 ? 1 : (pq == 4 ? 2 : 0);
            const int z = pq == 0 ? 0 : 1;
            auto mac = [&](uint4 a, uint4 b, f32x4 &c) __attribute__((always_inline)) {
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
            };
#pragma unroll
            for (int c = 0; c < NTC; ++c) mac(ha[0][p], hb[c][0][q], acc[0][z][c]);
#pragma unroll
            for (int c = 0; c < NTC; ++c) mac(ha[0][p], hb[c][1][q], acc[1][z][c]);
#pragma unroll
            for (int c = 0; c < NTC; ++c) mac(na[p], hb[c][1][q], acc[0][z][c]);
#pragma unroll
            for (int c = 0; c < NTC; ++c) mac(ha[1][p], hb[c][0][q], acc[1][z][c]);
        }
        if (--left == 0) {
            flush();
            left = every;
        }
    }
    flush();
    f32x4 accr[1][NTC], acci[1][NTC];
#pragma unroll
    for (int c = 0; c < NTC; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            accr[0][c][r] = (float)out[0][c][r];
            acci[0][c][r] = (float)out[1][c][r];
        }
    // The range, worked out anew from the thread's number, so that no register is
    // kept for it through the loop.  Bit j of `rows`: row j of B is full; a vector is
    // cnb rows, and B holds whole vectors.
    int l2 = threadIdx.x & 63;
    asm volatile("" : "+v"(l2));
    const int r2 = l2 & 15, o2 = loff(r2, l2 >> 4);
    const bool arow = i0 + r2 < g.M;
    const char *a2 = (const char *)g.A + (size_t)rb * brick_block_bytes(TNSLQ_FP32, g.nst) + loff(16 * r8 + r2, l2 >> 4);
    uint64_t rows = 0;
#pragma unroll
    for (int c = 0; c < NTC; ++c) {
        uint64_t m = pieces_full(bitsB[c]);
        m |= m >> 32;
        rows |= ((m | m >> 16) & 0xffffu) << (16 * c);
    }
    bool low = pieces_full(arow ? bitsA : 0) == 0 && arow && units_nonzero(a2, sbeg, send);
    const uint64_t all = g.N < 64 ? ((uint64_t)1 << g.N) - 1 : ~(uint64_t)0;
    if ((rows & all) != all) {
        const int cnb = 1 << (g.cnb_log2 < 6 ? g.cnb_log2 : 6);
        const uint64_t vec = cnb < 64 ? ((uint64_t)1 << cnb) - 1 : ~(uint64_t)0;
        for (int v = 0; v < g.N; v += cnb) {
            if (rows & vec << v) continue;
#pragma unroll
            for (int c = 0; c < NTC; ++c) {
                const int j = 16 * c + r2;
                if (j < g.N && vec << v >> j & 1) low = low || units_nonzero(gb + o2 + c * OC, sbeg, send);
            }
        }
    }
    if (__ballot(low) || nonfinite_tiles<TNSLQ_FP32, 1, NTC>(g, i0, 0, l2, accr, acci)) {
        const int pa[1] = {0};
        int pb[NTC];
#pragma unroll
        for (int c = 0; c < NTC; ++c) pb[c] = o2 + c * OC;
        plain_tiles<TNSLQ_FP32, 1, NTC>(a2, pa, gb, pb, sbeg, send, accr, acci);
    }
    store_tiles<TNSLQ_FP32, 1, NTC>(g, s, i0, 0, l2, accr, acci);
}

}  // namespace

hipError_t launch_gemm_thin(int prec, const GemmDesc &g, hipStream_t st) {
    const int64_t waves = (g.M + BM - 1) / BM * 8 * g.S;
    const int64_t nblocks = (waves + THIN_WAVES - 1) / THIN_WAVES;
    if (nblocks < 1 || nblocks > 0xffffff || (prec == TNSLQ_FP32 && g.N > 64)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)nblocks, (unsigned)((g.N + 63) / 64)), block(64 * THIN_WAVES);
    const int ntc = g.N <= 48 ? (int)((g.N + 15) / 16) : 4;
#define TNSLQ_THIN(C)                                                             \
    do {                                                                          \
        if (prec == TNSLQ_FP64)                                                   \
            hipLaunchKernelGGL((k_thin_product<C>), grid, block, 0, st, g);       \
        else                                                                      \
            hipLaunchKernelGGL((k_thin_fp32<C>), grid, block, 0, st, g);          \
    } while (0)
    switch (ntc) {
        case 1: TNSLQ_THIN(1); break;
        case 2: TNSLQ_THIN(2); break;
        case 3: TNSLQ_THIN(3); break;
        default: TNSLQ_THIN(4); break;
    }
#undef TNSLQ_THIN
    return hipGetLastError();
}

}  // namespace tnslq
