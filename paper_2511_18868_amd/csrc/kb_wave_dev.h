// Reductions over a wave by cross-lane moves (no LDS traffic).
#pragma once
#include "kb_internal.h"

namespace kb {

// Cross-lane steps inside rows of 16 lanes (data-parallel primitives: no LDS
// traffic): lanes 1,0,3,2 and 2,3,0,1 of every four, then mirrors inside every
// eight and every sixteen.  After the four steps every lane of a row holds the
// row's result; rows are combined through scalar registers.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = (int)(unsigned)b, hi = (int)(b >> 32);
    const unsigned lo2 = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const unsigned hi2 = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi2 << 32) | lo2));
}
__device__ __forceinline__ float row_max_f(float v) {
    v = fmaxf(v, dpp_f<0xB1>(v));
    v = fmaxf(v, dpp_f<0x4E>(v));
    v = fmaxf(v, dpp_f<0x141>(v));
    v = fmaxf(v, dpp_f<0x140>(v));
    return v;
}
__device__ __forceinline__ float row_min_f(float v) {
    v = fminf(v, dpp_f<0xB1>(v));
    v = fminf(v, dpp_f<0x4E>(v));
    v = fminf(v, dpp_f<0x141>(v));
    v = fminf(v, dpp_f<0x140>(v));
    return v;
}
// sum over the 16 lanes of a row, in a fixed order, delivered to all 16
__device__ __forceinline__ double row_sum_d(double v) {
    v += dpp_d<0xB1>(v);
    v += dpp_d<0x4E>(v);
    v += dpp_d<0x141>(v);
    v += dpp_d<0x140>(v);
    return v;
}
__device__ __forceinline__ float lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_d(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// (rows are combined by handing lane 15's value to the next row, then lane 31's to the upper half: two
// moves and one scalar read instead of four)
__device__ __forceinline__ float wave_max_f(float v) {
    v = row_max_f(v);
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x142, 0xa, 0xf, false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x143, 0xc, 0xf, false)));
    return lane_f(v, 63);
}
__device__ __forceinline__ float wave_min_f(float v) {
    v = row_min_f(v);
    return fminf(fminf(lane_f(v, 0), lane_f(v, 16)), fminf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ __forceinline__ double wave_max_d(double v) {
    v = fmax(v, dpp_d<0xB1>(v));
    v = fmax(v, dpp_d<0x4E>(v));
    v = fmax(v, dpp_d<0x141>(v));
    v = fmax(v, dpp_d<0x140>(v));
    return fmax(fmax(lane_d(v, 0), lane_d(v, 16)), fmax(lane_d(v, 32), lane_d(v, 48)));
}
// The lane that holds the largest value of the lanes with `has`, the lowest such lane on ties; -1:
// none has.  The values are numbers.  Rounded to fp32 they keep their order, so a lane that alone
// reaches the largest fp32 value is the one - a dozen instructions; only where several do (equal or
// nearly equal values) the fp64 values are compared.
__device__ __forceinline__ int wave_top_lane(double v, bool has) {
    const unsigned long long any = __ballot(has);
    if (!any) return -1;
    const float f = has ? (float)v : -INFINITY;
    const float m = wave_max_f(f);
    unsigned long long top = __ballot(has && f == m);
    if (top & (top - 1)) {
        const bool in = has && f == m;
        const double best = wave_max_d(in ? v : -INFINITY);
        top = __ballot(in && v == best);
    }
    return __ffsll((long long)top) - 1;
}
__device__ __forceinline__ int wave_min_i(int v) {
    auto step = [](int x, int y) { return x < y ? x : y; };
    v = step(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false));
    v = step(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false));
    v = step(v, __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false));
    v = step(v, __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false));
    return step(step(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                step(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ double wave_sum_d(double v) {
    v = row_sum_d(v);
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}

}  // namespace kb
