// The 16 x 16 tiles of the contraction kernels: fragments of brick rows, one
// reduction stage of the complex product in FP64, and the epilogue.
#pragma once
#include "operands.h"

namespace tnslq {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int BM = 128, BN = 128;
constexpr int ROWB = 64;                 // bytes per brick row
constexpr int TILEB = BM * ROWB;         // bytes per plane of a brick
static_assert(BM == BRICK_ROWS && BN == BRICK_ROWS && ROWB == BRICK_ROW_BYTES, "one brick per operand per step");

template <int PREC> struct MP;
template <> struct MP<TNSLQ_BF16X3> {
    static constexpr int NPL = 6;        // re_hi, re_lo, im_hi, im_lo, sum_hi, sum_lo
    using acc = f32x4;
};
template <> struct MP<TNSLQ_BF16X6> {
    static constexpr int NPL = 6;        // re_hi, re_mid, re_lo, im_hi, im_mid, im_lo
    using acc = f32x4;
};
template <> struct MP<TNSLQ_FP32> {
    static constexpr int NPL = 2;
    using acc = f32x4;
};
template <> struct MP<TNSLQ_FP64> {
    static constexpr int NPL = 2;
    using acc = f64x4;
};
// a 16-byte unit of a brick row feeds one 16x16x32 BF16 MFMA per lane, two of
// them one in FP32 (split in BF16 pieces), and one two 16x16x4 FP64 MFMAs
static_assert(brick_epr(TNSLQ_BF16X3) == 32 && brick_epr(TNSLQ_FP32) == 16 && brick_epr(TNSLQ_FP64) == 8,
              "brick rows of 64 bytes");
static_assert(MP<TNSLQ_BF16X3>::NPL == planes_of(TNSLQ_BF16X3) && MP<TNSLQ_BF16X6>::NPL == planes_of(TNSLQ_BF16X6) &&
                  MP<TNSLQ_FP32>::NPL == planes_of(TNSLQ_FP32) && MP<TNSLQ_FP64>::NPL == planes_of(TNSLQ_FP64),
              "planes per brick");

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ inline uint4 neg_bf16x8(uint4 v) {
    return make_uint4(v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u);
}
__device__ inline uint4 neg_f64x2(uint4 v) { return make_uint4(v.x, v.y ^ 0x80000000u, v.z, v.w ^ 0x80000000u); }
__device__ inline double f64_at(uint4 v, int t) {
    return t == 0 ? __hiloint2double((int)v.y, (int)v.x) : __hiloint2double((int)v.w, (int)v.z);
}

// byte offset of 16-byte unit `u` of staged row `row` within a plane tile
__device__ inline int loff(int row, int u) { return row * ROWB + 16 * (u ^ brick_swizzle(row)); }

// One FP64 reduction stage of the complex product for a wave's WTM x WTN tiles.
template <int WTM, int WTN>
__device__ __forceinline__ void stage_mfma(const uint4 (&fa)[WTM][2], const uint4 (&fb)[WTN][2],
                                           f64x4 (&accr)[WTM][WTN], f64x4 (&acci)[WTM][WTN]) {
    uint4 nai[WTM];
#pragma unroll
    for (int x = 0; x < WTM; ++x) nai[x] = neg_f64x2(fa[x][1]);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int a = 0; a < WTM; ++a)
#pragma unroll
            for (int b = 0; b < WTN; ++b) {
                const double ar = f64_at(fa[a][0], t), ai = f64_at(fa[a][1], t), nai_t = f64_at(nai[a], t);
                const double br = f64_at(fb[b][0], t), bi = f64_at(fb[b][1], t);
                accr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, accr[a][b], 0, 0, 0);
                accr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(nai_t, bi, accr[a][b], 0, 0, 0);
                acci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, acci[a][b], 0, 0, 0);
                acci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, acci[a][b], 0, 0, 0);
            }
}

// Epilogue of a wave's WTM x WTN tiles of 16 x 16 whose first output row and
// column are (wi0, wj0): output register r of lane l holds column l % 16 and
// row 4 (l / 16) + r (FP32 accumulators) or row 4 r + l / 16 (FP64); with SWAP
// (operands of the instruction exchanged) row l % 16 and column 4 (l / 16) + r.
template <int PREC, int WTM, int WTN, bool SWAP = false>
__device__ __forceinline__ void store_tiles(const GemmDesc &g, int s, int64_t wi0, int64_t wj0, int lane,
                                            const typename MP<PREC>::acc (&accr)[WTM][WTN],
                                            const typename MP<PREC>::acc (&acci)[WTM][WTN]) {
    const int frow = lane & 15, fk = lane >> 4;
    const int64_t cnb_mask = ((int64_t)1 << g.cnb_log2) - 1;
#pragma unroll
    for (int a = 0; a < WTM; ++a)
#pragma unroll
        for (int b = 0; b < WTN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int orow = PREC == TNSLQ_FP64 ? 4 * r + fk : 4 * fk + r;
                const int64_t i = wi0 + a * 16 + (SWAP ? frow : orow);
                const int64_t j = wj0 + b * 16 + (SWAP ? orow : frow);
                if (i >= g.M || j >= g.N) continue;
                const int64_t jq = j >> g.cnb_log2, jr = j & cnb_mask;
                const auto vr = accr[a][b][r], vi = acci[a][b][r];
                if (g.out_mode == 0) {
                    const int64_t row = jq * g.crs + (i & cnb_mask);
                    const int64_t col = (i & ~cnb_mask) + jr;
                    const int64_t idx = brick_index(PREC, g.c_nst, row, col);
                    if constexpr (PREC == TNSLQ_FP64)
                        store_planes<PREC>(g.C, brick_ps(PREC), idx, vr, vi);
                    else
                        store_planes_f<PREC>(g.C, brick_ps(PREC), idx, vr, vi);
                } else {
                    const int64_t addr = s * g.c_split + jq * g.cbs + i * g.ldc + jr;
                    if constexpr (PREC == TNSLQ_FP64)
                        ((double2 *)g.C)[addr] = make_double2(vr, vi);
                    else
                        ((float2 *)g.C)[addr] = make_float2(vr, vi);
                }
            }
}

}  // namespace
}  // namespace tnslq
