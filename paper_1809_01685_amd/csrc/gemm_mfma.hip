// Complex "NT" contraction C = A * B^T on the matrix cores (gfx950), for the
// two contractions of Sec. V Eq. 4, in these arithmetics:
//   BF16X3  operands split as hi + lo BF16 pieces, three products of pieces
//           per real product (hi*hi + hi*lo + lo*hi), v_mfma_f32_16x16x32_bf16,
//           FP32 accumulation (k_cgemm_bf16x3);
//   BF16X6  hi + mid + lo pieces, the six products of pieces (p, q) with
//           p + q < 3, FP32 accumulation restarted every 64 terms
//           (k_cgemm_bf16x6, 128 x 64 output tiles);
//   FP32    FP32 operands, split into three exact BF16 pieces on their way to
//           LDS, the same six products, FP32 accumulation in two levels
//           (k_cgemm_fp32);
//   FP64    v_mfma_f64_16x16x4_f64 (k_cgemm_fp64, 128 x 64 output tiles).
//
// A complex product takes three real ones (Gauss's form) but in BF16X6, which
// uses four, and in the FP32 and FP64 tiles that three do not reach (gemm_tiles.h):
//   Re C += Re A Re B + (-Im A) Im B,   Im C += Re A Im B + Im A Re B,
// the sign of Im A applied by flipping sign bits in registers.
//
// Tiling (wave64): a block of 8 waves computes a 128 x 128 (or 128 x 64)
// complex output tile, each wave 64 x 32 (32 x 32) in MFMA tiles of 16 x 16,
// two waves per SIMD so that one wave's LDS waits overlap the other's matrix
// instructions.  A brick of an operand is 128 rows x 64 bytes per plane (32
// BF16, 16 FP32 or 8 FP64 reduction terms); thread t copies bytes [16 t, 16 t
// + 16) of a plane, so each load instruction of the block reads 8 KiB of
// contiguous memory.  All but FP32 copy straight from global memory into LDS
// (global_load_lds_dwordx4: 16 bytes per lane, each wave 1 KiB of a plane
// tile).  Bricks store the four 16-byte units of a row XOR-swizzled by
// ((row >> 1) ^ (row >> 2)) & 3, so the fragment reads of 8 or 16 consecutive
// rows hit distinct banks.  Rows past the edge of C come from the bricks' row
// padding and their results are dropped; the reduction padding holds zeros.
// Each lane's 16-byte fragment feeds one BF16 MFMA (8 terms) or two FP64 MFMAs;
// A and B fragments pair the same reduction terms, so the order in which the
// terms of a unit enter the sum does not matter.
//
// Block order: the hardware deals blocks to the eight XCDs round robin, so
// block b is renumbered to give XCD b % 8 a contiguous range of output tiles,
// walked in groups of 4 tile rows; the ~32 blocks resident on one XCD then
// cover a compact 4 x 8 patch of tiles and share their A and B tiles in that
// XCD's L2.
#include "gemm_tiles.h"

#include <type_traits>

namespace tnslq {
namespace {

constexpr int GROUP_M = 4;
constexpr int WAVES_M = 2, WAVES_N = 4;
constexpr int TM = BM / (16 * WAVES_M), TN = BN / (16 * WAVES_N);
constexpr int NT = 64 * WAVES_M * WAVES_N;
static_assert(BM * ROWB / 16 == NT, "one 16-byte unit of every brick plane per thread");

// Output tile (i0, j0) and reduction split s of block b of nb (blockIdx.x of
// gridDim.x): the hardware deals blocks to the XCDs round robin, so block b is
// renumbered to give XCD b % 8 a contiguous range, walked in groups of GROUP_M
// tile rows.  In 32 bits (launches hold nb below 2^31): a 64-bit division is a
// microsecond of scalar code.
struct TileAt {
    int64_t i0, j0, sbeg, send;
    int s;
};
template <int TBN = BN>
__device__ inline TileAt tile_of(const GemmDesc &g, uint32_t b, uint32_t nb) {
    const uint32_t ntm = (uint32_t)((g.M + BM - 1) / BM), ntn = (uint32_t)((g.N + TBN - 1) / TBN);
    const uint32_t per_split = ntm * ntn;
    if (nb % 8 == 0) b = (b % 8) * (nb / 8) + b / 8;
    TileAt r;
    r.s = (int)(b / per_split);
    const uint32_t t = b % per_split;
    const uint32_t group = t / (GROUP_M * ntn), in_group = t % (GROUP_M * ntn);
    const uint32_t first_m = group * GROUP_M;
    const uint32_t gsize = ntm - first_m < GROUP_M ? ntm - first_m : GROUP_M;
    r.i0 = (int64_t)(first_m + in_group % gsize) * BM;
    r.j0 = (int64_t)(in_group / gsize) * TBN;
    const int64_t per = (uint32_t)g.nst / (uint32_t)g.S;
    r.sbeg = r.s * per;
    r.send = r.sbeg + per;
    return r;
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;
typedef __attribute__((address_space(1))) const char gbl_char_t;

template <int U, int END, typename F>
__device__ __forceinline__ void unroll_from(F &f) {
    if constexpr (U < END) {
        f(std::integral_constant<int, U>{});
        unroll_from<U + 1, END>(f);
    }
}

// ---------------------------------------------------------------------------
// FP64: three real products per complex product, as for BF16X3 below
//   T1 = sum Re A Re B,  T2 = sum Im A Im B,  T3 = sum (Re A + Im A)(Re B + Im B),
//   Re C = T1 - T2,      Im C = T3 - T1 - T2,
// a quarter fewer v_mfma_f64_16x16x4f64 than four; the sums Re + Im are formed
// from the fragments in registers (8 additions per 24 matrix instructions).
// T1 and T3 restart every two steps (16 terms), together, and are added into
// accumulators of their own.  Together, so that a real state and real vectors
// (T2 = 0, T3's terms T1's) give imaginary parts of exactly zero, as four products
// do; every 16 terms, so that the sums round less than a run of 64 terms in four
// products whatever is real (two operands real, state real, vectors real, none):
// 2.2, 3.2, 3.7, 4.1e-16 of the result against 80-bit sums where four products had
// 3.7, 3.8, 4.6, 5.4e-16 (restarts every 32 terms 2.8, 4.0, 4.3, 4.6; T3's alone 5.3,
// 4.7, 4.9, 4.9).  Their additions, on the matrix instructions' own FP64 units, are 3%
// of the time; a non-finite tile goes to four products (gemm_tiles.h).
// FP64 is bound by the matrix cores alone (a fragment read feeds six matrix
// instructions of 64 cycles), so the tile is chosen for the number of blocks:
// 128 x 64 outputs, 8 waves of 32 x 32 (2 x 2 tiles, 160 accumulator registers;
// 64 x 32 would take 320).  A step is one brick of A and half a brick of B
// (24 KiB), copied straight into a ring of four LDS buffers, four steps ahead;
// fragments of the next step are read between the current step's matrix
// instructions; one barrier per step.  Buffers and register sets are chosen at
// compile time (the loop body is four steps; what is left of a run, up to three,
// follows it without copies or barriers).  A 22-qubit block matvec of 5 vectors
// took 1575 us with 128 x 128 tiles of four products and 2048 splits' worth of
// partial sums, 690 with this.
constexpr int D_BN = 64, D_WAVES_N = 2, D_TM = 2, D_TN = 2, D_BODY = 4;

__global__ void __launch_bounds__(NT, 1) k_cgemm_fp64(GemmDesc g) {
    stamp(g.start);
    constexpr int NPL = 2, ABRICK = NPL * TILEB, BHALF = TILEB / 2, BSTEP = NPL * BHALF;
    __shared__ __attribute__((aligned(16))) char lA0[ABRICK], lA1[ABRICK], lA2[ABRICK], lA3[ABRICK];
    __shared__ __attribute__((aligned(16))) char lB0[BSTEP], lB1[BSTEP], lB2[BSTEP], lB3[BSTEP];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / D_WAVES_N, wn = wid % D_WAVES_N;
    const TileAt tl = tile_of<D_BN>(g, blockIdx.x, gridDim.x);
    const int64_t p0 = tl.sbeg, pend = tl.send, plast = pend - 1;
    const size_t blk = brick_block_bytes(TNSLQ_FP64, g.nst);
    const char *gA = (const char *)g.A + (size_t)(tl.i0 / BM) * blk;
    // B's rows j0 .. j0 + 63: the first or second half of every plane tile
    const char *gB = (const char *)g.B + (size_t)(tl.j0 / BN) * blk + ((tl.j0 % BN) / D_BN) * BHALF;
    const int w = __builtin_amdgcn_readfirstlane(wid);
    const uint32_t l16 = 16u * (uint32_t)lane;
    auto bufA = [&](auto bb) -> char * {
        constexpr int B = decltype(bb)::value;
        return B == 0 ? lA0 : (B == 1 ? lA1 : (B == 2 ? lA2 : lA3));
    };
    auto bufB = [&](auto bb) -> char * {
        constexpr int B = decltype(bb)::value;
        return B == 0 ? lB0 : (B == 1 ? lB1 : (B == 2 ? lB2 : lB3));
    };
    // copy step st (the last one again past the end): wave w takes KiB w of
    // both planes of A, and quarter w % 4 of plane w / 4 of B
    auto dma = [&](int64_t st, auto bb) __attribute__((always_inline)) {
        const int64_t q = st <= plast ? st : plast;
        gbl_char_t *pa = (gbl_char_t *)(gA + q * ABRICK + 1024 * w), *pa1 = pa + TILEB;
        gbl_char_t *pb = (gbl_char_t *)(gB + q * ABRICK + (w >> 2) * TILEB + (w & 3) * 1024);
        char *As = bufA(bb) + 1024 * w, *Bs = bufB(bb) + 1024 * w;
        // (the bases stay in scalar registers)
        asm volatile("" : "+s"(pa), "+s"(pa1), "+s"(pb));
        __builtin_amdgcn_global_load_lds((gbl_void_t *)(pa + l16), (lds_void_t *)As, 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gbl_void_t *)(pa1 + l16), (lds_void_t *)(As + TILEB), 16, 0, 0);
        __builtin_amdgcn_global_load_lds((gbl_void_t *)(pb + l16), (lds_void_t *)Bs, 16, 0, 0);
    };
    const int frow = lane & 15, fk = lane >> 4;
    // (rows 16 apart have their units in the same order)
    const int oa = loff(wm * D_TM * 16 + frow, fk), ob = loff(wn * D_TN * 16 + frow, fk);
    uint4 fa[2][D_TM][NPL], fb[2][D_TN][NPL];
    auto rd = [&](auto ss, auto bb) __attribute__((always_inline)) {
        constexpr int S = decltype(ss)::value;
        const char *As = bufA(bb), *Bs = bufB(bb);
#pragma unroll
        for (int x = 0; x < D_TM; ++x)
#pragma unroll
            for (int p = 0; p < NPL; ++p) fa[S][x][p] = *(const uint4 *)(As + p * TILEB + oa + x * 16 * ROWB);
#pragma unroll
        for (int x = 0; x < D_TN; ++x)
#pragma unroll
            for (int p = 0; p < NPL; ++p) fb[S][x][p] = *(const uint4 *)(Bs + p * BHALF + ob + x * 16 * ROWB);
    };
    // sums of the current chunk (T2's of all), and T1's and T3's of the chunks before
    f64x4 t[3][D_TM][D_TN], t1[D_TM][D_TN], t3[D_TM][D_TN];
#pragma unroll
    for (int a = 0; a < D_TM; ++a)
#pragma unroll
        for (int b = 0; b < D_TN; ++b) t[0][a][b] = t[1][a][b] = t[2][a][b] = t1[a][b] = t3[a][b] = f64x4{0, 0, 0, 0};
    auto restart = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < D_TM; ++a)
#pragma unroll
            for (int b = 0; b < D_TN; ++b) {
                t1[a][b] += t[0][a][b];
                t3[a][b] += t[2][a][b];
                t[0][a][b] = t[2][a][b] = f64x4{0, 0, 0, 0};
            }
    };
    // the products of fragment set C
    auto products = [&](auto cc) __attribute__((always_inline)) {
        constexpr int C = decltype(cc)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int a = 0; a < D_TM; ++a)
#pragma unroll
                    for (int b = 0; b < D_TN; ++b) {
                        const double ar = f64_at(fa[C][a][0], h), ai = f64_at(fa[C][a][1], h);
                        const double br = f64_at(fb[C][b][0], h), bi = f64_at(fb[C][b][1], h);
                        t[q][a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            q == 0 ? ar : (q == 1 ? ai : ar + ai), q == 0 ? br : (q == 1 ? bi : br + bi), t[q][a][b], 0, 0,
                            0);
                    }
    };
    int64_t base = p0;
    auto step = [&](auto uu) __attribute__((always_inline)) {
        constexpr int U = decltype(uu)::value, C = U % 2;
        constexpr std::integral_constant<int, C> cc{};
        rd(std::integral_constant<int, C ^ 1>{}, std::integral_constant<int, (U + 1) % 4>{});
        dma(base + U + 4, std::integral_constant<int, U>{});
        products(cc);
        // 2 MFMA, 8 x (LDS read, MFMA), 3 x (copy, MFMA), 11 MFMA
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 11, 0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0076);   // vmcnt(6): step st + 2 landed; lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (U % 2 == 1) {
            restart();
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    dma(p0, std::integral_constant<int, 0>{});
    dma(p0 + 1, std::integral_constant<int, 1>{});
    dma(p0 + 2, std::integral_constant<int, 2>{});
    dma(p0 + 3, std::integral_constant<int, 3>{});
    __builtin_amdgcn_s_waitcnt(0x0f79);   // vmcnt(9): step p0 landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    rd(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    __builtin_amdgcn_s_waitcnt(0x0076);   // vmcnt(6): step p0 + 1 landed; lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    for (; base + D_BODY <= pend; base += D_BODY) unroll_from<0, D_BODY>(step);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // the last steps and the copies past the end, before LDS is given up
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (base < pend) {
        products(std::integral_constant<int, 0>{});
        if (base + 1 < pend) {
            rd(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
            products(std::integral_constant<int, 1>{});
            restart();
            if (base + 2 < pend) {
                rd(std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
                products(std::integral_constant<int, 0>{});
            }
        }
    }
    restart();

    f64x4 accr[D_TM][D_TN], acci[D_TM][D_TN];
#pragma unroll
    for (int a = 0; a < D_TM; ++a)
#pragma unroll
        for (int b = 0; b < D_TN; ++b) {
            accr[a][b] = t1[a][b] - t[1][a][b];
            acci[a][b] = t3[a][b] - t1[a][b] - t[1][a][b];
        }
    // worked out anew from what the loop keeps: no registers for it through the loop
    int l2 = threadIdx.x & 63;
    asm volatile("" : "+v"(l2));
    const int m2 = w / D_WAVES_N * D_TM * 16, n2 = w % D_WAVES_N * D_TN * 16;
    if (nonfinite_tiles<TNSLQ_FP64, D_TM, D_TN>(g, tl.i0 + m2, tl.j0 + n2, (int)l2, accr, acci)) {
        // T3, or a sum Re + Im, may be infinite where the result is not (gemm_tiles.h)
        int pa[D_TM], pb[D_TN];
#pragma unroll
        for (int x = 0; x < D_TM; ++x) pa[x] = loff(m2 + x * 16 + (l2 & 15), l2 >> 4);
#pragma unroll
        for (int x = 0; x < D_TN; ++x) pb[x] = loff(n2 + x * 16 + (l2 & 15), l2 >> 4);
        plain_tiles<TNSLQ_FP64, D_TM, D_TN>(gA, pa, gB, pb, tl.sbeg, tl.send, accr, acci);
    }
    asm volatile("" : "+v"(l2));   // nor for the stores' addresses through this one
    store_tiles<TNSLQ_FP64, D_TM, D_TN>(g, tl.s, tl.i0 + m2, tl.j0 + n2, (int)l2, accr, acci);
}

hipError_t launch_fp64(const GemmDesc &g, hipStream_t st) {
    const int64_t nblocks = ((g.M + BM - 1) / BM) * ((g.N + D_BN - 1) / D_BN) * g.S;
    if (nblocks < 1 || nblocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_cgemm_fp64, dim3((unsigned)nblocks), dim3(NT), 0, st, g);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP32 on the BF16 matrix cores: an FP32 value is the exact sum of three BF16
// pieces (8 + 8 + 8 significant bits), a product of two values the six
// products of pieces (p, q) with p + q < 3 up to 2^-26 of it, and BF16
// instructions run at 16 times the rate of v_mfma_f32_16x16x4f32; with three
// real products per complex product a term costs 18 BF16 instructions where
// the FP32 unit took 16 times 4 (18 / 64 of the time).  The operands stay FP32 bricks: a
// step of 32 terms (two bricks) is loaded into registers, split there (a
// packed conversion, its widening and a subtraction per pair and piece) and
// written to LDS as three BF16 planes, so that memory and L2 see 8 bytes per
// value and not 18.
// Sums: each of T1, T2, T3 is accumulated over FP32_CHUNK steps (256 terms, or
// what GemmDesc::chunk says) in matrix-core accumulators that start from zero,
// the products of leading pieces apart from the five small ones (an addition
// rounds at the size of the sum, so adding those five to it rounds six times as
// often: 5.2e-7 instead of 2.0e-7 at 22 qubits), then added into Re C and Im C;
// T1, T2 and T3 take turns on one set of accumulators.  Error of a block matvec
// against 64 bits: 1.1e-7 to 2.2e-7 of the result from 10 to 24 qubits, where the
// FP32 unit with sums restarted every 64 terms had 2.0e-7 to 3.3e-7.
// Values that the pieces do not reach, and sums that overflow, go to the FP32
// unit (gemm_tiles.h): 1% of the time at 26 qubits, 2% at 22, for the test.
// Block, waves and tiles as k_cgemm_bf16x3: 128 x 128 outputs, 8 waves of
// 64 x 32; 48 matrix instructions per wave and step for 18 fragment reads.  Two
// LDS buffers (96 KiB), one barrier per step: the step after next is loaded, the
// next one split and written, then the current one's matrix instructions run.
// 26 qubits (65536 x 8192 outputs over 1024 terms): 34.0 to 22.2 ms, 130 to 198
// TFLOP/s.  Bound by the split and the loads ahead of each step's matrix
// instructions: interleaving them needs registers (it spilled 220), and giving
// the two waves of a SIMD alternate phases took 23.7 ms.
constexpr int FP32_CHUNK = 8;   // steps of 32 terms per restart

__global__ void __launch_bounds__(NT, 1) k_cgemm_fp32(GemmDesc g) {
    stamp(g.start);
    constexpr int FBRICK = 2 * TILEB;   // an FP32 brick: re, im
    constexpr int BUF = 3 * TILEB;      // an operand's three BF16 planes of a step
    __shared__ __attribute__((aligned(16))) char lds[2][2][BUF];
    __shared__ int some_low;   // a row of the tile held no value that the pieces reach
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;
    const TileAt tl = tile_of(g, blockIdx.x, gridDim.x);
    const size_t blk = brick_block_bytes(TNSLQ_FP32, g.nst);
    const char *gA = (const char *)g.A + (size_t)(tl.i0 / BM) * blk + 16 * tid;
    const char *gB = (const char *)g.B + (size_t)(tl.j0 / BN) * blk + 16 * tid;
    const int nsteps = (int)((tl.send - tl.sbeg + 1) / 2), chunk = g.chunk ? g.chunk : FP32_CHUNK;
    // thread t holds unit t % 4 of row t / 4 of a brick plane: four terms, 8
    // bytes of a BF16 row, in its first half (first brick) or second
    const int srow = tid >> 2, su = (tid & 3) ^ brick_swizzle(srow);
    const int so0 = loff(srow, su >> 1) + 8 * (su & 1), so1 = loff(srow, 2 + (su >> 1)) + 8 * (su & 1);

    // (chunk of steps from c0, product q, step s of the chunk)
    struct Cursor {
        int c0, q, s;
    };
    auto advance = [&](Cursor &c) __attribute__((always_inline)) {
        const int len = min(chunk, nsteps - c.c0);
        if (++c.s == len) {
            c.s = 0;
            if (++c.q == 3) {
                c.q = 0;
                c.c0 += chunk;
            }
        }
    };
    // staged values: [operand][brick of the step]; a second set for T3
    float4 v[2][2], v2[2][2];
    auto load = [&](const Cursor &c) __attribute__((always_inline)) {
        if (c.c0 >= nsteps) return;
        const int64_t st = tl.sbeg + 2 * (int64_t)(c.c0 + c.s);
        const int64_t o0 = st * FBRICK + (c.q == 1 ? TILEB : 0);
        const bool two = st + 1 < tl.send;
        v[0][0] = *(const float4 *)(gA + o0);
        v[1][0] = *(const float4 *)(gB + o0);
        // a last odd brick: the step's second half is zeros
        v[0][1] = two ? *(const float4 *)(gA + o0 + FBRICK) : make_float4(0.f, 0.f, 0.f, 0.f);
        v[1][1] = two ? *(const float4 *)(gB + o0 + FBRICK) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (c.q == 2) {
            v2[0][0] = *(const float4 *)(gA + o0 + TILEB);
            v2[1][0] = *(const float4 *)(gB + o0 + TILEB);
            v2[0][1] = two ? *(const float4 *)(gA + o0 + FBRICK + TILEB) : make_float4(0.f, 0.f, 0.f, 0.f);
            v2[1][1] = two ? *(const float4 *)(gB + o0 + FBRICK + TILEB) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto split2 = [&](float x, float y, uint32_t (&h)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const bf16x2 b = __builtin_convertvector((f32x2{x, y}), bf16x2);
            h[p] = __builtin_bit_cast(uint32_t, b);
            x -= __uint_as_float(h[p] << 16);
            y -= __uint_as_float(h[p] & 0xffff0000u);
        }
    };
    uint64_t full[2] = {0, 0};   // lanes that held a value of A, of B that the pieces reach (gemm_tiles.h)
    auto put = [&](int q, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            uint32_t bits = 0;   // of the leading pieces
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float4 x = v[o][h];
                if (q == 2) {
                    x.x += v2[o][h].x;
                    x.y += v2[o][h].y;
                    x.z += v2[o][h].z;
                    x.w += v2[o][h].w;
                }
                uint32_t a[3], b[3];
                split2(x.x, x.y, a);
                split2(x.z, x.w, b);
                bits |= a[0] | b[0];
                char *d = lds[buf][o] + (h ? so1 : so0);
#pragma unroll
                for (int p = 0; p < 3; ++p) *(uint2 *)(d + p * TILEB) = make_uint2(a[p], b[p]);
            }
            if (q != 2) full[o] |= pieces_full(bits);
        }
    };
    const int frow = lane & 15, fk = lane >> 4;
    // (rows 16 apart have their units in the same order)
    const int oa = loff(wm * TM * 16 + frow, fk), ob = loff(wn * TN * 16 + frow, fk);
    f32x4 t[TM][TN], tlow[TM][TN], accr[TM][TN], acci[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) t[a][b] = tlow[a][b] = accr[a][b] = acci[a][b] = f32x4{0, 0, 0, 0};

    if (tid == 0) some_low = 0;
    Cursor cur{0, 0, 0}, nxt{0, 0, 0}, ld{0, 0, 0};
    load(ld);
    advance(ld);
    put(0, 0);
    load(ld);
    nxt = ld;
    advance(ld);
    __syncthreads();
    const int total = 3 * nsteps;
    int buf = 0;
    for (int i = 0; i < total; ++i, buf ^= 1) {
        const char *As = lds[buf][0], *Bs = lds[buf][1];
        uint4 fa[TM][3], fb[TN][3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int x = 0; x < TM; ++x) fa[x][p] = *(const uint4 *)(As + p * TILEB + oa + x * 16 * ROWB);
#pragma unroll
            for (int x = 0; x < TN; ++x) fb[x][p] = *(const uint4 *)(Bs + p * TILEB + ob + x * 16 * ROWB);
        }
        if (i + 1 < total) put(nxt.q, buf ^ 1);
        nxt = ld;
        load(ld);
        advance(ld);
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) {
            // (0,0), (0,1), (1,0), (1,1), (0,2), (2,0): pieces in the order they are read
            const int p = pq == 2 || pq == 3 ? 1 : (pq == 5 ? 2 : 0);
            const int q = pq == 1 || pq == 3 ? 1 : (pq == 4 ? 2 : 0);
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    f32x4 &c = pq == 0 ? t[a][b] : tlow[a][b];
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[a][p]), as_bf16x8(fb[b][q]), c, 0, 0, 0);
                }
        }
        const int q = cur.q;
        advance(cur);
        if (cur.q != q || cur.s == 0) {
            // the chunk's sum of product q
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    t[a][b] += tlow[a][b];
                    if (q == 0) {
                        accr[a][b] += t[a][b];
                        acci[a][b] -= t[a][b];
                    } else if (q == 1) {
                        accr[a][b] -= t[a][b];
                        acci[a][b] -= t[a][b];
                    } else {
                        acci[a][b] += t[a][b];
                    }
                    t[a][b] = tlow[a][b] = f32x4{0, 0, 0, 0};
                }
        }
        __syncthreads();
    }
    // The range (gemm_tiles.h), worked out anew from the thread's number, so that no
    // register is kept for it through the loop.  Wave w holds rows 16 w .. 16 w + 15
    // of an operand, four lanes each.
    int t2 = tid;
    asm volatile("" : "+v"(t2));
    const int l2 = t2 & 63, r2 = t2 >> 2, m2 = (t2 >> 6) / WAVES_N, n2 = (t2 >> 6) % WAVES_N;
    const char *bA = (const char *)g.A + (size_t)(tl.i0 / BM) * blk, *bB = (const char *)g.B + (size_t)(tl.j0 / BN) * blk;
    const bool have[2] = {tl.i0 + r2 < g.M, tl.j0 + r2 < g.N};
    const uint64_t arows = __ballot(have[0]), brows = __ballot(have[1]);
    if (((full[0] & arows) != arows || (full[1] & brows) != brows) && l2 == 0) some_low = 1;
    __syncthreads();
    bool low = some_low;
    if (low) {
        low = false;
        uint64_t *waves = (uint64_t *)lds;   // [operand][wave]
        if (l2 == 0) {
            waves[t2 >> 6] = full[0] & arows;
            waves[8 + (t2 >> 6)] = full[1] & brows;
        }
        __syncthreads();
#pragma unroll 1
        for (int o = 0; o < 2; ++o) {
            // the rows of this thread's group: all of A's, those of one vector (cnb) of B's
            const int group = o == 0 || g.cnb_log2 > 6 ? BM : 1 << g.cnb_log2;
            uint64_t m = 0;
            if (group >= 16)
                for (int w = (r2 & -group) / 16; w < ((r2 & -group) + group) / 16; ++w) m |= waves[8 * o + w];
            else
                m = waves[8 * o + r2 / 16] >> (4 * (r2 & 15 & -group)) & (((uint64_t)1 << (4 * group)) - 1);
            if (m == 0 && (o == 0 ? have[0] : have[1]))
                low = low || units_nonzero((o == 0 ? bA : bB) + 16 * t2, tl.sbeg, tl.send);
        }
        low = __syncthreads_or(low);
    }
    const int64_t wi0 = tl.i0 + m2 * TM * 16, wj0 = tl.j0 + n2 * TN * 16;
    if (low || nonfinite_tiles<TNSLQ_FP32, TM, TN>(g, wi0, wj0, l2, accr, acci)) {
        int pa[TM], pb[TN];
#pragma unroll
        for (int x = 0; x < TM; ++x) pa[x] = loff(m2 * TM * 16 + x * 16 + (l2 & 15), l2 >> 4);
#pragma unroll
        for (int x = 0; x < TN; ++x) pb[x] = loff(n2 * TN * 16 + x * 16 + (l2 & 15), l2 >> 4);
        plain_tiles<TNSLQ_FP32, TM, TN>(bA, pa, bB, pb, tl.sbeg, tl.send, accr, acci);
    }
    store_tiles<TNSLQ_FP32, TM, TN>(g, tl.s, wi0, wj0, l2, accr, acci);
}

hipError_t launch_fp32(const GemmDesc &g, hipStream_t st) {
    const int64_t nblocks = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * g.S;
    if (nblocks < 1 || nblocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_cgemm_fp32, dim3((unsigned)nblocks), dim3(NT), 0, st, g);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BF16X3: three real products per complex product (Gauss's form),
//   T1 = sum Re A Re B,  T2 = sum Im A Im B,  T3 = sum (Re A + Im A)(Re B + Im B),
//   Re C = T1 - T2,      Im C = T3 - T1 - T2,
// each real product split as hi*hi + hi*lo + lo*hi: 9 matrix instructions per
// pair of 16 x 16 tiles and reduction step instead of 12.  The operands carry
// Re + Im as a third pair of planes (operands.h), so a brick is three 16 KiB
// pairs (re, im, sum; hi and lo of 128 rows each) in the order of the three
// products.  Staging a whole brick of both operands twice would take 192 KiB
// of LDS; the kernel stages instead one pair of planes of each operand per
// "phase" (32 KiB), and the phases of a block's run of bricks are consecutive
// 16 KiB pieces of its rows of A and of B.  Same block, waves and tiles as
// k_cgemm_fp32 (128 x 128 outputs, 8 waves of 64 x 32); per phase a wave
// issues 24 matrix instructions into the accumulators of that phase's product.
// Pipeline over a ring of four LDS buffers (128 KiB): in phase ph the matrix
// instructions run on phase ph's fragments while, issued between them, a wave
// reads phase ph + 1's fragments from its buffer into the second register set
// and the block copies phase ph + 4 into the buffer phase ph has left (its
// fragments are in registers); one barrier ends the phase once phase ph + 2
// has landed (the copies of ph + 3 and ph + 4 stay in flight).  Issuing the
// reads and copies before the matrix instructions instead left the matrix
// cores idle after every barrier: 254 / 270 ms per launch against 244 / 244.
// The barrier is a bare s_barrier after explicit wait counts: __syncthreads
// would add a fence that waits for every copy in flight.  Buffers, register
// sets and accumulators are chosen at
// compile time (the LDS buffers are eight arrays, so that the compiler tells a
// fragment read of one buffer from a copy into another): the loop body is 12
// phases (4 bricks), and a run whose phase count is not a multiple of 12
// starts with the last 3, 6 or 9 phases of that body, so the loop itself has
// no branch (a branch around each phase's instructions cost 8%).  Against the
// four-product kernel on the 30-qubit contractions, launched alone on one box:
// 244 / 244 ms per launch against 283 / 282, 14% rather than 25%, the rest
// taken by the 1.5x bytes staged per step (with the copies left out the loop
// took 189 ms) and the power they cost under the chip's power limit.
// Runs of up to X3_WALK bricks: a block per CU walks its tiles, and past a
// tile's last phase the copies go on with the next tile's first four, in flight
// through the tile's stores, so that a tile does not start with empty buffers
// (where its phases are a multiple of the loop body; others start anew): 65536 x
// 8192 outputs over 256 terms 3040 to 2930 us, 508 to 496 us over 1024 terms of
// a 22-qubit state.  Longer runs take a block per tile: their start is 1 us in
// 65, and blocks dealt as CUs come free keep neighbouring tiles together (a
// 28-qubit estimate, 65536 x 32768 over 4096 terms and back, took 1525 ms walked
// and 1482 dealt).
constexpr int PHB = 2 * TILEB;    // one pair of planes of one operand: 16 KiB
constexpr int X3_BODY = 12;       // phases per loop iteration: lcm(2 sets, 3 products, 4 buffers)
constexpr int X3_BLOCKS = 256;    // one per CU
constexpr int X3_WALK = 32;

__global__ void __launch_bounds__(NT, 1) k_cgemm_bf16x3(GemmDesc g) {
    stamp(g.start);
    __shared__ __attribute__((aligned(16))) char lA0[PHB], lA1[PHB], lA2[PHB], lA3[PHB];
    __shared__ __attribute__((aligned(16))) char lB0[PHB], lB1[PHB], lB2[PHB], lB3[PHB];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / WAVES_N, wn = wid % WAVES_N;
    // the block's tiles: blockIdx.x, blockIdx.x + gridDim.x, ..
    const uint32_t ntiles = (uint32_t)((g.M + BM - 1) / BM * ((g.N + BN - 1) / BN) * g.S);
    const size_t blk = brick_block_bytes(TNSLQ_BF16X3, g.nst);
    TileAt tl = tile_of(g, blockIdx.x, ntiles);
    // phases of the tile's run of bricks (3 per brick), as many in every tile
    const int64_t np = 3 * (tl.send - tl.sbeg);
    const char *gA = (const char *)g.A + (size_t)(tl.i0 / BM) * blk + 3 * tl.sbeg * PHB;
    const char *gB = (const char *)g.B + (size_t)(tl.j0 / BN) * blk + 3 * tl.sbeg * PHB;
    // what follows the run: the next tile's first phases, or the last phase again
    const char *nA = gA, *nB = gB;
    const int u0 = (int)((X3_BODY - (uint32_t)np % X3_BODY) % X3_BODY);
    const bool seam = u0 == 0;
    const uint32_t toff = 16u * (uint32_t)tid;
    const int wofs = 1024 * __builtin_amdgcn_readfirstlane(wid);
    auto bufA = [&](auto bb) -> char * {
        constexpr int B = decltype(bb)::value;
        return B == 0 ? lA0 : (B == 1 ? lA1 : (B == 2 ? lA2 : lA3));
    };
    auto bufB = [&](auto bb) -> char * {
        constexpr int B = decltype(bb)::value;
        return B == 0 ? lB0 : (B == 1 ? lB1 : (B == 2 ? lB2 : lB3));
    };
    // copy phase ph into buffer bb: thread t copies bytes [16 t, 16 t + 16) of
    // both plane tiles of A and of B
    auto dma = [&](int64_t ph, auto bb) __attribute__((always_inline)) {
        const bool past = ph >= np;
        const int64_t q = !past ? ph : (seam ? ph - np : np - 1);
        const char *pa = (past ? nA : gA) + q * PHB, *pb = (past ? nB : gB) + q * PHB;
        char *As = bufA(bb) + wofs, *Bs = bufB(bb) + wofs;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            __builtin_amdgcn_global_load_lds((gbl_void_t *)(pa + p * TILEB + toff), (lds_void_t *)(As + p * TILEB), 16,
                                             0, 0);
            __builtin_amdgcn_global_load_lds((gbl_void_t *)(pb + p * TILEB + toff), (lds_void_t *)(Bs + p * TILEB), 16,
                                             0, 0);
        }
    };
    const int frow = lane & 15, fk = lane >> 4;
    int oa[TM], ob[TN];
#pragma unroll
    for (int x = 0; x < TM; ++x) oa[x] = loff(wm * TM * 16 + x * 16 + frow, fk);
#pragma unroll
    for (int x = 0; x < TN; ++x) ob[x] = loff(wn * TN * 16 + x * 16 + frow, fk);
    // fragments (hi, lo) of the wave's A and B tiles, two sets
    uint4 fa[2][TM][2], fb[2][TN][2];
    auto rd = [&](auto ss, auto bb) __attribute__((always_inline)) {
        constexpr int S = decltype(ss)::value;
        const char *As = bufA(bb), *Bs = bufB(bb);
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int p = 0; p < 2; ++p) fa[S][x][p] = *(const uint4 *)(As + p * TILEB + oa[x]);
#pragma unroll
        for (int x = 0; x < TN; ++x)
#pragma unroll
            for (int p = 0; p < 2; ++p) fb[S][x][p] = *(const uint4 *)(Bs + p * TILEB + ob[x]);
    };
    // T1, T2, T3
    f32x4 t[3][TM][TN];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) t[q][a][b] = f32x4{0, 0, 0, 0};

    // phase base + U of the loop body (U = 0 .. 11): fragments in set U % 2,
    // operands in buffer U % 4, product U % 3
    int64_t base = 0;
    auto phase = [&](auto uu) __attribute__((always_inline)) {
        constexpr int U = decltype(uu)::value;
        constexpr int C = U % 2, Q = U % 3;
        const int64_t ph = base + U;
        rd(std::integral_constant<int, C ^ 1>{}, std::integral_constant<int, (U + 1) % 4>{});
        dma(ph + 4, std::integral_constant<int, U % 4>{});
#pragma unroll
        for (int term = 0; term < 3; ++term) {
            const int p = term == 2 ? 1 : 0, q = term == 1 ? 1 : 0;
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b)
                    // B first: a lane's four outputs are then one row's
                    t[Q][a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fb[C][b][q]), as_bf16x8(fa[C][a][p]),
                                                                         t[Q][a][b], 0, 0, 0);
        }
        // the matrix instructions start right after the barrier, the 12
        // fragment reads and the 4 copies issued one between each pair
        // (2 MFMA, then 12 x (LDS read, MFMA), 4 x (copy, MFMA), 6 MFMA)
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0078);   // vmcnt(8): phase ph + 2 landed; lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // the run starts at body position U0 (0, 3, 6 or 9), so that it ends with
    // a whole body: phases 0 .. 3 into buffers U0 .. U0 + 3 (mod 4), phase 0's
    // fragments into set U0 % 2, then body positions U0 .. 11
    auto start = [&](auto u0) __attribute__((always_inline)) {
        constexpr int V = decltype(u0)::value;
        dma(0, std::integral_constant<int, V % 4>{});
        dma(1, std::integral_constant<int, (V + 1) % 4>{});
        dma(2, std::integral_constant<int, (V + 2) % 4>{});
        dma(3, std::integral_constant<int, (V + 3) % 4>{});
        __builtin_amdgcn_s_waitcnt(0x0f7c);   // vmcnt(12): phase 0 landed
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        rd(std::integral_constant<int, V % 2>{}, std::integral_constant<int, V % 4>{});
        __builtin_amdgcn_s_waitcnt(0x0078);   // vmcnt(8): phase 1 landed; lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        base = -V;
        unroll_from<V, X3_BODY>(phase);
        base += X3_BODY;
    };
    // Output as bricks (the first contraction's intermediary).  A lane holds
    // four columns of one row per tile: 8 bytes of a plane.  Exchanging the
    // odd 16 lanes of the first column tile with the even ones of the second
    // gives every lane 8 consecutive columns, a 16-byte unit when cnb >= 8 (8
    // consecutive reduction terms of one brick row), and the wave 16 rows of 32
    // columns: rows i of one environment index are rows of the same brick, so
    // a store is 1 KiB of consecutive bytes of a plane.  65536 x 8192 outputs
    // over 256 terms, where a tile's output weighs as much as its 24 phases:
    // 4350 us with rows of 2-byte writes into LDS and roundings in integers,
    // 3380 through LDS in 8-byte writes, 3040 this way, without LDS or barriers.
    auto store_bricks = [&](const TileAt &tl, int lane, const f32x4 (&accr)[TM][TN], const f32x4 (&acci)[TM][TN])
                            __attribute__((always_inline)) {
        const int frow = lane & 15, fk = lane >> 4;
        static_assert(TN == 2, "32 columns: a brick row");
        constexpr int64_t PS = brick_ps(TNSLQ_BF16X3);
        const int64_t cnb_mask = ((int64_t)1 << g.cnb_log2) - 1;
        const int64_t j = tl.j0 + wn * TN * 16 + 16 * (fk & 1) + 8 * (fk >> 1);
        const int64_t jrow = (j >> g.cnb_log2) * g.crs, jcol = j & cnb_mask;
#pragma unroll
        for (int a = 0; a < TM; ++a) {
            const int64_t i = tl.i0 + wm * TM * 16 + a * 16 + frow;
            uint16_t *out = (uint16_t *)g.C + brick_index(TNSLQ_BF16X3, g.c_nst, jrow + (i & cnb_mask), (i & ~cnb_mask) + jcol);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                uint32_t h[TN][2][2];   // tile, piece, pair of columns
#pragma unroll
                for (int b = 0; b < TN; ++b) {
                    const f32x4 re = accr[a][b], im = acci[a][b];
                    const f32x4 v = q == 0 ? re : (q == 1 ? im : re + im);
                    split_bf16_pair(v[0], v[1], h[b][0][0], h[b][1][0]);
                    split_bf16_pair(v[2], v[3], h[b][0][1], h[b][1][1]);
                }
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const auto x = __builtin_amdgcn_permlane16_swap(h[0][p][0], h[1][p][0], false, false);
                    const auto y = __builtin_amdgcn_permlane16_swap(h[0][p][1], h[1][p][1], false, false);
                    if (i < g.M && j < g.N) *(uint4 *)(out + (2 * q + p) * PS) = make_uint4(x[0], y[0], x[1], y[1]);
                }
            }
        }
    };

    for (uint32_t at = blockIdx.x;; at += gridDim.x) {
        const bool last = at + gridDim.x >= ntiles;
        TileAt next = tl;
        if (!last) {
            next = tile_of(g, at + gridDim.x, ntiles);
            nA = (const char *)g.A + (size_t)(next.i0 / BM) * blk + 3 * next.sbeg * PHB;
            nB = (const char *)g.B + (size_t)(next.j0 / BN) * blk + 3 * next.sbeg * PHB;
        } else {
            nA = gA;
            nB = gB;
        }
        if (seam && at != blockIdx.x) {
            // phases 0 and 1 are there, 2 and 3 on their way; phase 0's
            // fragments again, rather than held through the last tile's stores
            rd(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            base = 0;
        } else {
            switch (u0) {
                case 3: start(std::integral_constant<int, 3>{}); break;
                case 6: start(std::integral_constant<int, 6>{}); break;
                case 9: start(std::integral_constant<int, 9>{}); break;
                default: start(std::integral_constant<int, 0>{}); break;
            }
        }
        for (; base < np; base += X3_BODY) unroll_from<0, X3_BODY>(phase);
        if (last || !seam) {
            // no copy outlives the block, and none is in a buffer that start() fills
            __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
        f32x4 accr[TM][TN], acci[TM][TN];
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                accr[a][b] = t[0][a][b] - t[1][a][b];
                acci[a][b] = t[2][a][b] - t[0][a][b] - t[1][a][b];
            }
        // the addresses of the stores are worked out here, not kept in registers
        // through the next tile
        int elane = lane;
        asm volatile("" : "+v"(elane));
        if (g.out_mode != 0 || g.cnb_log2 < 3) {
            store_tiles<TNSLQ_BF16X3, TM, TN, true>(g, tl.s, tl.i0 + wm * TM * 16, tl.j0 + wn * TN * 16, elane, accr, acci);
        } else {
            store_bricks(tl, elane, accr, acci);
        }
        if (last) break;
        tl = next;
        gA = nA;
        gB = nB;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int a = 0; a < TM; ++a)
#pragma unroll
                for (int b = 0; b < TN; ++b) t[q][a][b] = f32x4{0, 0, 0, 0};
    }
}

hipError_t launch_bf16x3(const GemmDesc &g, hipStream_t st) {
    const int64_t ntiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * g.S;
    if (ntiles < 1 || ntiles > 0x7fffffff) return hipErrorInvalidConfiguration;
    const int64_t nblocks = g.nst / g.S <= X3_WALK ? std::min<int64_t>(ntiles, X3_BLOCKS) : ntiles;
    hipLaunchKernelGGL(k_cgemm_bf16x3, dim3((unsigned)nblocks), dim3(NT), 0, st, g);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BF16X6: operands split as hi + mid + lo BF16 pieces (six planes per
// operand), the products of pieces (p, q) with p + q < 3, six per real
// product, in FP32 on the matrix cores.  Six planes of a 128 x 128 tile would
// take 96 KiB of LDS per step, so a block computes 128 x 64 outputs: A's
// brick (48 KiB) and the half of B's brick that holds its 64 rows (24 KiB)
// per step, double buffered in 144 KiB.  Eight waves (two per SIMD), each
// 32 x 32 outputs (2 x 2 tiles of 16 x 16): per step a wave issues 96 MFMAs,
// as in the three-piece kernel.  The matrix-core sums restart every two steps
// (64 terms) and are added into a second FP32 accumulator, so that no FP32
// running sum grows past 64 terms.
constexpr int X6_BN = 64, X6_WAVES_M = 4, X6_WAVES_N = 2;
constexpr int X6_TM = BM / (16 * X6_WAVES_M), X6_TN = X6_BN / (16 * X6_WAVES_N);
constexpr int X6_NT = 64 * X6_WAVES_M * X6_WAVES_N;
constexpr int X6_FLUSH = 2;
static_assert(X6_TM == 2 && X6_TN == 2 && X6_NT == 512, "32 x 32 per wave");

__global__ void __launch_bounds__(X6_NT, 1) k_cgemm_bf16x6(GemmDesc g) {
    stamp(g.start);
    constexpr int NPL = 6;
    constexpr int ABRICK = NPL * TILEB;        // A's brick, all planes: 48 KiB
    constexpr int BHALF = TILEB / 2;           // 64 rows of one plane of B: 4 KiB
    constexpr int BSTAGE = NPL * BHALF;        // 24 KiB
    __shared__ __attribute__((aligned(16))) char ldsA0[ABRICK], ldsA1[ABRICK], ldsB0[BSTAGE], ldsB1[BSTAGE];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int wm = wid / X6_WAVES_N, wn = wid % X6_WAVES_N;
    const TileAt tl = tile_of<X6_BN>(g, blockIdx.x, gridDim.x);
    const int64_t sbeg = tl.sbeg, send = tl.send;

    const size_t blk = brick_block_bytes(TNSLQ_BF16X6, g.nst);
    const char *gA = (const char *)g.A + (size_t)(tl.i0 / BM) * blk;
    // B's rows j0 .. j0 + 63: the first or second half of every plane tile
    const char *gB = (const char *)g.B + (size_t)(tl.j0 / BN) * blk + ((tl.j0 % BN) / X6_BN) * BHALF;
    const int w = __builtin_amdgcn_readfirstlane(wid);
    const uint32_t loff16 = 16u * (uint32_t)lane;
    // A: thread t copies bytes [16 t, 16 t + 16) of each plane tile; B: wave
    // w copies the 1 KiB pieces w, w + 8 and w + 16 of the 24 (plane piece / 4,
    // quarter piece % 4 of its 4 KiB)
    auto dma = [&](int64_t st, int buf) __attribute__((always_inline)) {
        const char *pa = gA + st * ABRICK, *pb = gB + st * ABRICK;
        char *As = (buf ? ldsA1 : ldsA0) + 1024 * w, *Bs = buf ? ldsB1 : ldsB0;
#pragma unroll
        for (int p = 0; p < NPL; ++p)
            __builtin_amdgcn_global_load_lds((gbl_void_t *)(pa + p * TILEB + 1024 * w + loff16),
                                             (lds_void_t *)(As + p * TILEB), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int piece = w + 8 * i, plane = piece / 4, quarter = piece % 4;
            __builtin_amdgcn_global_load_lds((gbl_void_t *)(pb + plane * TILEB + quarter * 1024 + loff16),
                                             (lds_void_t *)(Bs + plane * BHALF + quarter * 1024), 16, 0, 0);
        }
    };
    const int frow = lane & 15, fk = lane >> 4;
    int oa[X6_TM], ob[X6_TN];
#pragma unroll
    for (int x = 0; x < X6_TM; ++x) oa[x] = loff(wm * X6_TM * 16 + x * 16 + frow, fk);
#pragma unroll
    for (int x = 0; x < X6_TN; ++x) ob[x] = loff(wn * X6_TN * 16 + x * 16 + frow, fk);

    f32x4 accr[X6_TM][X6_TN], acci[X6_TM][X6_TN], outr[X6_TM][X6_TN], outi[X6_TM][X6_TN];
#pragma unroll
    for (int a = 0; a < X6_TM; ++a)
#pragma unroll
        for (int b = 0; b < X6_TN; ++b) {
            accr[a][b] = acci[a][b] = outr[a][b] = outi[a][b] = f32x4{0, 0, 0, 0};
        }
    const int64_t last = send - 1;
    dma(sbeg, 0);
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    __syncthreads();
    int nstage = 0;
    for (int64_t st = sbeg; st < send; ++st) {
        const int buf = (int)((st - sbeg) & 1);
        const char *As = buf ? ldsA1 : ldsA0, *Bs = buf ? ldsB1 : ldsB0;
        uint4 fa[X6_TM][NPL], fb[X6_TN][NPL];
#pragma unroll
        for (int x = 0; x < X6_TM; ++x)
#pragma unroll
            for (int p = 0; p < NPL; ++p) fa[x][p] = *(const uint4 *)(As + p * TILEB + oa[x]);
#pragma unroll
        for (int x = 0; x < X6_TN; ++x)
#pragma unroll
            for (int p = 0; p < NPL; ++p) fb[x][p] = *(const uint4 *)(Bs + p * BHALF + ob[x]);
        // every fragment read of the step is issued before the copy into
        // the other buffer
        __builtin_amdgcn_sched_barrier(0);
        dma(st + 1 <= last ? st + 1 : last, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        // pieces (p, q) with p + q < 3; Re C += Re A Re B + (-Im A) Im B,
        // Im C += Re A Im B + Im A Re B
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) {
            const int p = pq < 3 ? 0 : (pq < 5 ? 1 : 2);
            const int q = pq < 3 ? pq : (pq < 5 ? pq - 3 : 0);
#pragma unroll
            for (int a = 0; a < X6_TM; ++a) {
                const uint4 na = neg_bf16x8(fa[a][3 + p]);
#pragma unroll
                for (int b = 0; b < X6_TN; ++b) {
                    accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[a][p]), as_bf16x8(fb[b][q]),
                                                                          accr[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[a][p]),
                                                                          as_bf16x8(fb[b][3 + q]), acci[a][b], 0, 0, 0);
                    accr[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(na), as_bf16x8(fb[b][3 + q]),
                                                                          accr[a][b], 0, 0, 0);
                    acci[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fa[a][3 + p]),
                                                                          as_bf16x8(fb[b][q]), acci[a][b], 0, 0, 0);
                }
            }
        }
        if (++nstage == X6_FLUSH) {
#pragma unroll
            for (int a = 0; a < X6_TM; ++a)
#pragma unroll
                for (int b = 0; b < X6_TN; ++b) {
                    outr[a][b] += accr[a][b];
                    outi[a][b] += acci[a][b];
                    accr[a][b] = acci[a][b] = f32x4{0, 0, 0, 0};
                }
            nstage = 0;
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) and lgkmcnt(0)
        __syncthreads();
    }
    if (nstage) {
#pragma unroll
        for (int a = 0; a < X6_TM; ++a)
#pragma unroll
            for (int b = 0; b < X6_TN; ++b) {
                outr[a][b] += accr[a][b];
                outi[a][b] += acci[a][b];
            }
    }
    store_tiles<TNSLQ_BF16X6, X6_TM, X6_TN>(g, tl.s, tl.i0 + wm * X6_TM * 16, tl.j0 + wn * X6_TN * 16, lane, outr,
                                            outi);
}

hipError_t launch_bf16x6(const GemmDesc &g, hipStream_t st) {
    const int64_t nblocks = ((g.M + BM - 1) / BM) * ((g.N + X6_BN - 1) / X6_BN) * g.S;
    if (nblocks < 1 || nblocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_cgemm_bf16x6, dim3((unsigned)nblocks), dim3(X6_NT), 0, st, g);
    return hipGetLastError();
}

template <int PREC>
bool supported(const GemmDesc &g) {
    if (thin_product(PREC, g.M, g.N, g.S, g.nst)) return ((uintptr_t)g.A % 16) == 0 && ((uintptr_t)g.B % 16) == 0;
    return g.S >= 1 && g.nst % g.S == 0 && ((uintptr_t)g.A % 16) == 0 && ((uintptr_t)g.B % 16) == 0;
}

}  // namespace

// Whether the matrix-core kernel takes this contraction: BF16X3, BF16X6, FP32
// or FP64 bricks, the bricks divided evenly between the splits.
bool gemm_mfma_supported(int prec, const GemmDesc &g) {
    switch (prec) {
        case TNSLQ_BF16X3: return supported<TNSLQ_BF16X3>(g);
        case TNSLQ_BF16X6: return supported<TNSLQ_BF16X6>(g);
        case TNSLQ_FP32: return supported<TNSLQ_FP32>(g);
        case TNSLQ_FP64: return supported<TNSLQ_FP64>(g);
        default: return false;
    }
}

hipError_t launch_gemm_mfma(int prec, const GemmDesc &g, hipStream_t st) {
    if (thin_product(prec, g.M, g.N, g.S, g.nst))
        return launch_gemm_thin(prec, g, st);
    switch (prec) {
        case TNSLQ_BF16X3: return launch_bf16x3(g, st);
        case TNSLQ_BF16X6: return launch_bf16x6(g, st);
        case TNSLQ_FP32: return launch_fp32(g, st);
        case TNSLQ_FP64: return launch_fp64(g, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tnslq
