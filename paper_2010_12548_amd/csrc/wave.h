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

// v of lane (lane ^ M), M a power of two below 64, in the vector ALU: moves
// inside rows of 16 lanes, then swaps of rows and of halves.  A cross-lane
// read through LDS takes about five times as long.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "");
    if constexpr (M == 1) return dpp0<0xb1, 0xf>(v);        // quads 1 0 3 2
    else if constexpr (M == 2) return dpp0<0x4e, 0xf>(v);   // quads 2 3 0 1
    else if constexpr (M == 4) {
        // lanes 4-7 and 12-15 of a row from four lanes before, the others after
        const int up = __builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xa, false);
        return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)v, 0x104, 0xf, 0x5, false);
    } else if constexpr (M == 8) return dpp0<0x128, 0xf>(v);  // rows rotated by 8
    else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    }
}

template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v)
{
    return (uint64_t)lane_xor<M>((uint32_t)v) | (uint64_t)lane_xor<M>((uint32_t)(v >> 32)) << 32;
}
