// Wave64 helpers on registers: sums over a wave by data-parallel-primitive
// moves, in a fixed order, and uniform reads of one lane.
#pragma once
#include <hip/hip_runtime.h>

namespace tnslq {

// v's DPP-moved copy (both 32-bit halves moved alike); 0 in lanes of rows
// outside ROWS and in those without a source
template <int CTRL, int ROWS>
__device__ inline double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int CTRL, int ROWS>
__device__ inline double dpp_add(double v) {
    return v + dpp_move<CTRL, ROWS>(v);
}

// lane `lane`'s value (uniform `lane`), in every lane
__device__ inline double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The sum over the wave's 64 lanes, returned to every lane: pairs, quads,
// half rows and rows of 16 by lane permutations within a row, then rows 0-1
// into row 1 and rows 0-3 into row 3 by row broadcasts; lane 63 holds the
// total.  A fixed order, done in registers.
__device__ inline double wave_total(double v) {
    v = dpp_add<0xB1, 0xf>(v);    // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E, 0xf>(v);    // quad_perm [2, 3, 0, 1]
    v = dpp_add<0x141, 0xf>(v);   // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);   // row_mirror
    v = dpp_add<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return lane_value(v, 63);
}

// The same sum in the order of a shuffle-down tree: lanes 32 apart, then 16, 8,
// 4, 2 and 1, returned to every lane.
__device__ inline double wave_tree_total(double v) {
    auto halves = [](double x, auto swap) {
        const long long b = __double_as_longlong(x);
        const auto lo = swap((unsigned)b), hi = swap((unsigned)(b >> 32));
        return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
               __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
    };
    v = halves(v, [](unsigned u) { return __builtin_amdgcn_permlane32_swap(u, u, false, false); });
    v = halves(v, [](unsigned u) { return __builtin_amdgcn_permlane16_swap(u, u, false, false); });
    v = dpp_add<0x128, 0xf>(v);   // row_ror:8
    v = dpp_add<0x124, 0xf>(v);   // row_ror:4
    v = dpp_add<0x4E, 0xf>(v);    // quad_perm [2, 3, 0, 1]
    return dpp_add<0xB1, 0xf>(v);   // quad_perm [1, 0, 3, 2]
}

// Lane i: the largest of lanes 0 .. i, for values that are not negative (a NaN
// counts as nothing, as with fmax).
__device__ inline double wave_scan_max(double v) {
    v = fmax(v, dpp_move<0x111, 0xf>(v));   // row_shr:1, 2, 4, 8
    v = fmax(v, dpp_move<0x112, 0xf>(v));
    v = fmax(v, dpp_move<0x114, 0xf>(v));
    v = fmax(v, dpp_move<0x118, 0xf>(v));
    v = fmax(v, dpp_move<0x142, 0xa>(v));   // row_bcast:15 into rows 1 and 3
    return fmax(v, dpp_move<0x143, 0xc>(v));   // row_bcast:31 into rows 2 and 3
}

}  // namespace tnslq
