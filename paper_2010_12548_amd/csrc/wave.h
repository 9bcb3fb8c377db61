// Scans over a wavefront's 64 lanes in the vector ALU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// v from the lane that the DPP control names, 0 where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp0(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp0(uint64_t v)
{
    return (uint64_t)dpp0<CTRL, ROWS>((uint32_t)v) |
           (uint64_t)dpp0<CTRL, ROWS>((uint32_t)(v >> 32)) << 32;
}

struct OpAdd {
    template <typename T>
    __device__ static T f(T a, T b) { return a + b; }
};
struct OpMax {
    template <typename T>
    __device__ static T f(T a, T b) { return a > b ? a : b; }
};

// inclusive scan over the wavefront (identity 0; every lane takes part):
// shifts of 1, 2, 4, 8 inside the rows of 16 lanes, then the rows' last lanes
// broadcast, all in the vector ALU; a chain of six cross-lane reads through
// LDS takes ten times as long
template <typename OP>
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v = OP::f(v, dpp0<0x111, 0xf>(v));
    v = OP::f(v, dpp0<0x112, 0xf>(v));
    v = OP::f(v, dpp0<0x114, 0xf>(v));
    v = OP::f(v, dpp0<0x118, 0xf>(v));
    v = OP::f(v, dpp0<0x142, 0xa>(v));
    v = OP::f(v, dpp0<0x143, 0xc>(v));
    return v;
}

template <typename OP>
__device__ __forceinline__ uint64_t wave_scan(uint64_t v)
{
    v = OP::f(v, dpp0<0x111, 0xf>(v));
    v = OP::f(v, dpp0<0x112, 0xf>(v));
    v = OP::f(v, dpp0<0x114, 0xf>(v));
    v = OP::f(v, dpp0<0x118, 0xf>(v));
    v = OP::f(v, dpp0<0x142, 0xa>(v));
    v = OP::f(v, dpp0<0x143, 0xc>(v));
    return v;
}
