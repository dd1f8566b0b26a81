// The 16 x 16 tiles of the contraction kernels: fragments of brick rows, a
// reduction stage of the complex product in four real ones, the range that the
// three-product and split forms leave to it, and the epilogue.
#pragma once
#include <float.h>

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
__device__ inline uint4 neg_f32x4(uint4 v) {
    return make_uint4(v.x ^ 0x80000000u, v.y ^ 0x80000000u, v.z ^ 0x80000000u, v.w ^ 0x80000000u);
}
__device__ inline double f64_at(uint4 v, int t) {
    return t == 0 ? __hiloint2double((int)v.y, (int)v.x) : __hiloint2double((int)v.w, (int)v.z);
}
__device__ inline float f32_at(uint4 v, int t) {
    return __uint_as_float(t == 0 ? v.x : (t == 1 ? v.y : (t == 2 ? v.z : v.w)));
}

// byte offset of 16-byte unit `u` of staged row `row` within a plane tile
__device__ inline int loff(int row, int u) { return row * ROWB + 16 * (u ^ brick_swizzle(row)); }

// One reduction stage (a brick of each operand) of the complex product in four
// real ones for a wave's WTM x WTN tiles: FP64 or FP32 matrix instructions.
template <int PREC, int WTM, int WTN>
__device__ __forceinline__ void stage_mfma(const uint4 (&fa)[WTM][2], const uint4 (&fb)[WTN][2],
                                           typename MP<PREC>::acc (&accr)[WTM][WTN],
                                           typename MP<PREC>::acc (&acci)[WTM][WTN]) {
    static_assert(PREC == TNSLQ_FP64 || PREC == TNSLQ_FP32, "real and imaginary planes");
    uint4 nai[WTM];
#pragma unroll
    for (int x = 0; x < WTM; ++x) nai[x] = PREC == TNSLQ_FP64 ? neg_f64x2(fa[x][1]) : neg_f32x4(fa[x][1]);
#pragma unroll
    for (int t = 0; t < brick_epu(PREC); ++t)
#pragma unroll
        for (int a = 0; a < WTM; ++a)
#pragma unroll
            for (int b = 0; b < WTN; ++b) {
                if constexpr (PREC == TNSLQ_FP64) {
                    const double ar = f64_at(fa[a][0], t), ai = f64_at(fa[a][1], t), nai_t = f64_at(nai[a], t);
                    const double br = f64_at(fb[b][0], t), bi = f64_at(fb[b][1], t);
                    accr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, accr[a][b], 0, 0, 0);
                    accr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(nai_t, bi, accr[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, acci[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, acci[a][b], 0, 0, 0);
                } else {
                    const float ar = f32_at(fa[a][0], t), ai = f32_at(fa[a][1], t), nai_t = f32_at(nai[a], t);
                    const float br = f32_at(fb[b][0], t), bi = f32_at(fb[b][1], t);
                    accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, br, accr[a][b], 0, 0, 0);
                    accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(nai_t, bi, accr[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, bi, acci[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(ai, br, acci[a][b], 0, 0, 0);
                }
            }
}

// What the split and three-product forms leave out.  An FP32 value is the sum of
// three BF16 pieces only down to 2^-110: the last piece of a smaller one is
// below BF16's subnormals.  The sum of a value's real and imaginary part, and
// T3, reach infinity up to four times before the result does, and infinite
// terms give NaN (Inf - Inf) where four products give Inf.  So a tile whose
// operand (A's rows, or B's rows of one vector) is all below 2^-95 but not zero,
// or that has a non-finite output, is worked out again by plain_tiles.  FP32,
// vectors of 1e-36: 2.9e-7 of the result where the pieces are off by 1.3e-4.
// 2^-95 and not 2^-110, where the pieces' error passes the FP32 unit's, because
// "an exponent of 32 or more" is a test on the leading pieces' bits ORed
// together (maxima of the values took 50 registers more).

__device__ inline uint32_t or_bits(uint4 x) { return (x.x | x.y) | (x.z | x.w); }
// the lanes with a leading piece of 2^-95 or more (or an infinity or a NaN, which
// reach the output) among those whose bits are in m
__device__ inline uint64_t pieces_full(uint32_t m) { return __ballot((m & 0x70007000u) != 0); }
// whether the units at p (one per plane) of bricks [sbeg, send) hold a value
// other than zero.  Four bricks' loads in flight: a 26-qubit state with mostly
// zero rows (GHZ) takes 293 ms, with one brick 322, without zeros 266
__device__ inline bool units_nonzero(const char *p, int64_t sbeg, int64_t send) {
    uint32_t m = 0;
#pragma unroll 4
    for (int64_t st = sbeg; st < send; ++st)
#pragma unroll
        for (int q = 0; q < 2; ++q) m |= or_bits(*(const uint4 *)(p + (2 * st + q) * TILEB));
    return (m & 0x7fffffffu) != 0;
}

// Whether a wave's tiles hold a non-finite output (rows below M, columns below
// N: the padding's are dropped); layout as for store_tiles.
template <int PREC, int WTM, int WTN>
__device__ __forceinline__ bool nonfinite_tiles(const GemmDesc &g, int64_t wi0, int64_t wj0, int lane,
                                                const typename MP<PREC>::acc (&accr)[WTM][WTN],
                                                const typename MP<PREC>::acc (&acci)[WTM][WTN]) {
    using T = decltype(accr[0][0][0] + 0);
    T z = 0;   // NaN from the first infinity or NaN on
#pragma unroll
    for (int a = 0; a < WTM; ++a)
#pragma unroll
        for (int b = 0; b < WTN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) z = fma((T)acci[a][b][r], (T)0, fma((T)accr[a][b][r], (T)0, z));
    if (__ballot(z != 0) == 0) return false;
    // the padding's do not count
    const int frow = lane & 15, fk = lane >> 4;
    bool bad = false;
#pragma unroll
    for (int a = 0; a < WTM; ++a)
#pragma unroll
        for (int b = 0; b < WTN; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t i = wi0 + a * 16 + (PREC == TNSLQ_FP64 ? 4 * r + fk : 4 * fk + r), j = wj0 + b * 16 + frow;
                if (i < g.M && j < g.N && !(isfinite(accr[a][b][r]) && isfinite(acci[a][b][r]))) bad = true;
            }
    return __ballot(bad) != 0;
}

// A wave's tiles over bricks [sbeg, send) in four real products of the
// precision's own matrix instructions, sums restarted every four bricks; row
// tile a's fragments at ga + oa[a], column tile b's at gb + ob[b], from memory.
template <int PREC, int WTM, int WTN>
__device__ __forceinline__ void plain_tiles(const char *ga, const int (&oa)[WTM], const char *gb, const int (&ob)[WTN],
                                            int64_t sbeg, int64_t send, typename MP<PREC>::acc (&outr)[WTM][WTN],
                                            typename MP<PREC>::acc (&outi)[WTM][WTN]) {
    using Acc = typename MP<PREC>::acc;
    constexpr int BRICKB = 2 * TILEB;
#pragma unroll
    for (int a = 0; a < WTM; ++a)
#pragma unroll
        for (int b = 0; b < WTN; ++b) outr[a][b] = outi[a][b] = Acc{0, 0, 0, 0};
    for (int64_t s0 = sbeg; s0 < send; s0 += 4) {
        Acc accr[WTM][WTN], acci[WTM][WTN];
#pragma unroll
        for (int a = 0; a < WTM; ++a)
#pragma unroll
            for (int b = 0; b < WTN; ++b) accr[a][b] = acci[a][b] = Acc{0, 0, 0, 0};
#pragma unroll 1
        for (int64_t st = s0; st < send && st < s0 + 4; ++st) {
            uint4 fa[WTM][2], fb[WTN][2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
#pragma unroll
                for (int a = 0; a < WTM; ++a) fa[a][p] = *(const uint4 *)(ga + st * BRICKB + p * TILEB + oa[a]);
#pragma unroll
                for (int b = 0; b < WTN; ++b) fb[b][p] = *(const uint4 *)(gb + st * BRICKB + p * TILEB + ob[b]);
            }
            stage_mfma<PREC, WTM, WTN>(fa, fb, accr, acci);
        }
#pragma unroll
        for (int a = 0; a < WTM; ++a)
#pragma unroll
            for (int b = 0; b < WTN; ++b) {
                outr[a][b] += accr[a][b];
                outi[a][b] += acci[a][b];
            }
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
