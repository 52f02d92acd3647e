// sidm_wave.hpp -- reductions over the lanes of a wave.
#pragma once

#include "sidm_internal.hpp"

namespace sidm {

#ifdef __HIPCC__
// v moved by a DPP control (rotations within rows of 16 lanes)
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Minimum / maximum over each row of 16 lanes, on every lane of the row.
__device__ inline double row_min(double v)
{
    v = fmin(v, dpp_f64<0x128>(v));   // row_ror:8
    v = fmin(v, dpp_f64<0x124>(v));
    v = fmin(v, dpp_f64<0x122>(v));
    return fmin(v, dpp_f64<0x121>(v));
}

__device__ inline double row_max(double v)
{
    v = fmax(v, dpp_f64<0x128>(v));
    v = fmax(v, dpp_f64<0x124>(v));
    v = fmax(v, dpp_f64<0x122>(v));
    return fmax(v, dpp_f64<0x121>(v));
}

// Sum over each row of 16 lanes, in the same order on every lane.
__device__ inline double row_sum(double v)
{
    v += dpp_f64<0x128>(v);
    v += dpp_f64<0x124>(v);
    v += dpp_f64<0x122>(v);
    return v + dpp_f64<0x121>(v);
}

// ... and over the rows of the wave (v uniform within each row).
__device__ inline double rows_min(double v)
{
    v = fmin(v, __shfl_xor(v, 16, 64));
    return fmin(v, __shfl_xor(v, 32, 64));
}

__device__ inline double rows_max(double v)
{
    v = fmax(v, __shfl_xor(v, 16, 64));
    return fmax(v, __shfl_xor(v, 32, 64));
}

__device__ inline double rows_sum(double v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// Maximum over the lanes of the wave (not NaN).
__device__ inline float lanes_max(float v)
{
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(
                     0, __float_as_int(v), 0x128, 0xF, 0xF, false)));   // row_ror:8
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xF, 0xF,
                                                            false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xF, 0xF,
                                                            false)));
    v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xF, 0xF,
                                                            false)));
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}

// Sum over the lanes up to and including this one.
__device__ inline int lanes_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

// Box (lo xyz, hi xyz) of the positions of the lanes with `in` set.
__device__ inline void lanes_box(bool in, double px, double py, double pz, double* o)
{
    o[0] = rows_min(row_min(in ? px : INFINITY));
    o[1] = rows_min(row_min(in ? py : INFINITY));
    o[2] = rows_min(row_min(in ? pz : INFINITY));
    o[3] = rows_max(row_max(in ? px : -INFINITY));
    o[4] = rows_max(row_max(in ? py : -INFINITY));
    o[5] = rows_max(row_max(in ? pz : -INFINITY));
}
#endif

}  // namespace sidm
