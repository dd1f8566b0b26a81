// Operand formats of the two contractions and the contraction launcher
// interface: precisions and their BF16 splits, plane stores, the brick layout
// of an operand, and the GEMM descriptor.  Everything the contraction kernels
// are compiled from, apart from their own source file and their tiles
// (gemm_tiles.h), is here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "tnslq.h"

namespace tnslq {

// ------------------------------------------------------------ precisions
// Pieces per real component and bytes per stored piece.
__host__ __device__ constexpr int pieces_of(int prec) {
    return prec == TNSLQ_BF16X6 ? 3 : (prec == TNSLQ_BF16X3 ? 2 : 1);
}
__host__ __device__ constexpr int piece_bytes(int prec) {
    return prec == TNSLQ_FP64 ? 8 : (prec == TNSLQ_FP32 ? 4 : 2);
}
// Planes per stored complex value: the pieces of the real part, then those of
// the imaginary part; split BF16 (BF16X3) also stores the pieces of their sum
// Re + Im, which its contraction needs for the three-product form of a complex
// product (planes re_hi, re_lo, im_hi, im_lo, sum_hi, sum_lo).
__host__ __device__ constexpr int planes_of(int prec) { return prec == TNSLQ_BF16X3 ? 6 : 2 * pieces_of(prec); }

// ------------------------------------------------------------ BF16 helpers
// Round-to-nearest-even FP32 -> BF16 bits (the packed conversion instruction,
// one for two values; written out in integers it was six instructions each,
// most of the time of an epilogue that splits its outputs).
__device__ inline uint16_t f32_to_bf16_rne(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// re + im as its two rounded operands give it, whatever they were computed from.
template <class T> __device__ inline T rounded_sum(T re, T im) {
#pragma clang fp contract(off)
    return re + im;
}

// Split an FP32 value into `np` BF16 pieces whose sum approximates it:
// piece 0 = bf16(x), piece 1 = bf16(x - piece0), piece 2 = bf16(rest).
// The pieces are those of the rounded value x: no product that made it is
// drawn into the differences.
template <int NP>
__device__ inline void split_bf16(float x, uint16_t *out) {
#pragma clang fp contract(off)
    float r = x;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        uint16_t h = f32_to_bf16_rne(r);
        out[p] = h;
        r = r - bf16_to_f32(h);
    }
}
// split_bf16<2> of two values, their pieces packed x first.
__device__ inline void split_bf16_pair(float x, float y, uint32_t &hi, uint32_t &lo) {
#pragma clang fp contract(off)
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
    const float rx = x - __uint_as_float(hi << 16), ry = y - __uint_as_float(hi & 0xffff0000u);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){rx, ry}, bf16x2));
}
// Split an FP64 value: the first piece is taken from the double directly so
// that the pieces capture the value to ~2^-8 per piece.
template <int NP>
__device__ inline void split_bf16_d(double x, uint16_t *out) {
#pragma clang fp contract(off)
    double r = x;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        uint16_t h = f32_to_bf16_rne((float)r);
        out[p] = h;
        r = r - (double)bf16_to_f32(h);
    }
}

// Store one complex value (re, im) into plane arrays at element index `idx`.
// `ps` is the plane stride in elements.  Accepts double inputs.  BF16X3 also
// stores the split of re + im (rounded once, from the inputs' precision).
template <int PREC>
__device__ inline void store_planes(void *base, int64_t ps, int64_t idx, double re, double im) {
    if constexpr (PREC == TNSLQ_FP64) {
        double *p = (double *)base;
        p[idx] = re;
        p[ps + idx] = im;
    } else if constexpr (PREC == TNSLQ_FP32) {
        float *p = (float *)base;
        p[idx] = (float)re;
        p[ps + idx] = (float)im;
    } else {
        constexpr int NP = pieces_of(PREC);
        uint16_t *p = (uint16_t *)base;
        uint16_t h[NP];
        split_bf16_d<NP>(re, h);
#pragma unroll
        for (int q = 0; q < NP; ++q) p[q * ps + idx] = h[q];
        split_bf16_d<NP>(im, h);
#pragma unroll
        for (int q = 0; q < NP; ++q) p[(NP + q) * ps + idx] = h[q];
        if constexpr (PREC == TNSLQ_BF16X3) {
            split_bf16_d<NP>(rounded_sum(re, im), h);
#pragma unroll
            for (int q = 0; q < NP; ++q) p[(2 * NP + q) * ps + idx] = h[q];
        }
    }
}
// Same for FP32 accumulator values (the first contraction's output).
template <int PREC>
__device__ inline void store_planes_f(void *base, int64_t ps, int64_t idx, float re, float im) {
    if constexpr (PREC == TNSLQ_FP64) {
        double *p = (double *)base;
        p[idx] = re;
        p[ps + idx] = im;
    } else if constexpr (PREC == TNSLQ_FP32) {
        float *p = (float *)base;
        p[idx] = re;
        p[ps + idx] = im;
    } else {
        constexpr int NP = pieces_of(PREC);
        uint16_t *p = (uint16_t *)base;
        uint16_t h[NP];
        split_bf16<NP>(re, h);
#pragma unroll
        for (int q = 0; q < NP; ++q) p[q * ps + idx] = h[q];
        split_bf16<NP>(im, h);
#pragma unroll
        for (int q = 0; q < NP; ++q) p[(NP + q) * ps + idx] = h[q];
        if constexpr (PREC == TNSLQ_BF16X3) {
            split_bf16<NP>(rounded_sum(re, im), h);
#pragma unroll
            for (int q = 0; q < NP; ++q) p[(2 * NP + q) * ps + idx] = h[q];
        }
    }
}

// ------------------------------------------------------------ bricks
// An R x Kr operand is cut into bricks of 128 rows by 64 bytes of the
// reduction index (32 BF16, 16 FP32 or 8 FP64 terms) per plane; a brick holds
// all planes of its piece of the matrix one after the other (8 KiB each, in
// the order of planes_of), and
// bricks run along the reduction index first, then over blocks of 128 rows.
// Within a brick row the four 16-byte units are stored XOR-swizzled by
// ((row >> 1) ^ (row >> 2)) & 3, the order in which the contraction kernel
// keeps them in LDS.  Rows are padded to a multiple of 128 and the reduction
// index to a whole brick; padding along the reduction index must hold zeros.
// One brick is what the contraction kernel stages per reduction step (split
// BF16: one pair of planes at a time), so its loads are contiguous blocks of
// 8 KiB or more.
constexpr int BRICK_ROWS = 128;
constexpr int BRICK_ROW_BYTES = 64;
constexpr int BRICK_PLANE_BYTES = BRICK_ROWS * BRICK_ROW_BYTES;

// reduction terms per brick row
__host__ __device__ constexpr int brick_epr(int prec) { return BRICK_ROW_BYTES / piece_bytes(prec); }
// distance between the planes of one brick, in elements
__host__ __device__ constexpr int64_t brick_ps(int prec) { return (int64_t)BRICK_ROWS * brick_epr(prec); }
// bricks along the reduction index
__host__ __device__ inline int64_t brick_stages(int prec, int64_t Kr) {
    return (Kr + brick_epr(prec) - 1) / brick_epr(prec);
}
__host__ __device__ inline int64_t brick_rows(int64_t R) { return (R + BRICK_ROWS - 1) / BRICK_ROWS * BRICK_ROWS; }
// bytes of one block of 128 rows, and of a whole R x Kr operand
__host__ __device__ inline size_t brick_block_bytes(int prec, int64_t nst) {
    return (size_t)nst * planes_of(prec) * BRICK_PLANE_BYTES;
}
__host__ __device__ inline size_t brick_bytes(int prec, int64_t R, int64_t Kr) {
    return (size_t)(brick_rows(R) / BRICK_ROWS) * brick_block_bytes(prec, brick_stages(prec, Kr));
}
__host__ __device__ inline int brick_swizzle(int64_t row) { return (int)(((row >> 1) ^ (row >> 2)) & 3); }
// Element index (plane 0) of entry (r, l) of an operand with nst bricks along
// the reduction index; plane p of the entry is at + p * brick_ps(prec).
__host__ __device__ inline int64_t brick_index(int prec, int64_t nst, int64_t r, int64_t l) {
    const int epr = brick_epr(prec), epu = epr / 4;
    const int64_t rr = r % BRICK_ROWS, st = l / epr, ll = l % epr;
    const int64_t u = (ll / epu) ^ brick_swizzle(rr);
    return (((r / BRICK_ROWS) * nst + st) * planes_of(prec) * BRICK_ROWS + rr) * epr + u * epu + ll % epu;
}

// The 16-byte units (one per plane) of brick_epu consecutive reduction terms
// v of one row, stored at element index idx (plane 0) of the unit's first
// term: what store_planes writes term by term, in whole units.
__host__ __device__ constexpr int brick_epu(int prec) { return 16 / piece_bytes(prec); }
template <int PREC>
__device__ inline void store_unit(void *base, int64_t idx, const double2 (&v)[brick_epu(PREC)]) {
    constexpr int EPU = brick_epu(PREC);
    constexpr int64_t PS = brick_ps(PREC);
    if constexpr (PREC == TNSLQ_FP64) {
        double *p = (double *)base + idx;
        *(double2 *)p = make_double2(v[0].x, v[1].x);
        *(double2 *)(p + PS) = make_double2(v[0].y, v[1].y);
    } else if constexpr (PREC == TNSLQ_FP32) {
        float *p = (float *)base + idx;
        *(float4 *)p = make_float4((float)v[0].x, (float)v[1].x, (float)v[2].x, (float)v[3].x);
        *(float4 *)(p + PS) = make_float4((float)v[0].y, (float)v[1].y, (float)v[2].y, (float)v[3].y);
    } else {
        constexpr int NP = pieces_of(PREC), NC = planes_of(PREC) / NP;   // re, im (and their sum)
        uint16_t *p = (uint16_t *)base + idx;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint32_t w[NP][EPU / 2];
#pragma unroll
            for (int t = 0; t < EPU; ++t) {
                uint16_t h[NP];
                split_bf16_d<NP>(c == 0 ? v[t].x : (c == 1 ? v[t].y : rounded_sum(v[t].x, v[t].y)), h);
#pragma unroll
                for (int q = 0; q < NP; ++q) w[q][t / 2] = t % 2 ? w[q][t / 2] | (uint32_t)h[q] << 16 : h[q];
            }
#pragma unroll
            for (int q = 0; q < NP; ++q)
                *(uint4 *)(p + (c * NP + q) * PS) = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
        }
    }
}

// ------------------------------------------------------------ times
// The device's constant-rate clock, written by the first thread of a kernel's
// first block as it starts (p null: not asked for).  The phases of an estimate
// are timed by these instead of events around them: an event costs a launch's
// time on the stream, and small estimates are launches.
__device__ inline void stamp(uint64_t *p) {
    if (p && (blockIdx.x | blockIdx.y | blockIdx.z | threadIdx.x) == 0) *p = wall_clock64();
}

// ------------------------------------------------------------ GEMM
// C = A * B^T over complex brick operands: A is M x Kr, B is N x Kr, both with
// nst bricks along the reduction index and A, B pointing at their first block
// of rows.  The reduction is split into S equal runs of bricks.  With
// cnb = 2^cnb_log2, output element (i, j) of split s goes
//   out_mode 0: into a brick operand with c_nst bricks along its reduction
//               index, at row (j / cnb) * crs + i % cnb and reduction index
//               (i / cnb) * cnb + j % cnb (S = 1);
//   out_mode 1: to interleaved accumulator-type complex values at
//               s * c_split + (j / cnb) * cbs + i * ldc + j % cnb.
struct GemmDesc {
    const void *A;
    const void *B;
    void *C;
    int64_t M, N, Kr, nst;
    int S;
    int out_mode;
    int cnb_log2;
    int64_t crs, c_nst;
    int64_t ldc, cbs, c_split;
    uint64_t *start;   // where the kernel stamps its start, or null
    int chunk;         // FP32: steps of 32 terms per restarted sum, 0 for the kernel's own choice
};

// Whether an M x N product over nst bricks in S splits runs in 16-row tiles
// against up to 64 columns (k_thin_fp32, k_thin_product) instead of 128-row tiles:
//   FP32 up to 64 columns, where a 128-column tile is at least half padding (at
//     65 to 128 columns the large tile's reuse of A through LDS is worth the
//     padding);
//   FP64 up to 64 columns, a column tile of k_cgemm_fp64, which issues three
//     products to the four here but needs more rows to fill the chip: at 64
//     columns n = 864 takes 19 us a product here and 48 there, 2048 44 and 46,
//     4096 154 and 142, a 22-qubit block matvec 204 and 197;
//   FP64 over at most four bricks (32 terms), where four real products round less
//     than three (10 qubits: 3.73e-16 of the result against 4.18e-16) and the
//     matrix cores are not the bound.
// Its splits need not divide the bricks.
__host__ inline bool thin_product(int prec, int64_t M, int64_t N, int S, int64_t nst) {
    if ((prec != TNSLQ_FP32 && prec != TNSLQ_FP64) || S < 1 || (M + 127) / 128 * 2 * S > 0xffffff) return false;
    return N <= 64 || (prec == TNSLQ_FP64 && nst <= 4 * (int64_t)S && (N + 63) / 64 <= 65535);
}

hipError_t launch_gemm(int prec, const GemmDesc &g, hipStream_t st);
hipError_t launch_gemm_valu(int prec, const GemmDesc &g, hipStream_t st);
hipError_t launch_gemm_thin(int prec, const GemmDesc &g, hipStream_t st);
bool gemm_mfma_supported(int prec, const GemmDesc &g);
hipError_t launch_gemm_mfma(int prec, const GemmDesc &g, hipStream_t st);

}  // namespace tnslq
