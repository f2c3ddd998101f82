// Operations across the 64 lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace irgs {

// v of another lane (data-parallel primitive Ctrl); `old` in the lanes that have no source.
template <int Ctrl>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v)
{
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(static_cast<int>(old), static_cast<int>(v), Ctrl, 0xf, 0xf, false));
}

// Inclusive sum over the lanes.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v)
{
    v += dpp<0x111>(0u, v);
    v += dpp<0x112>(0u, v);
    v += dpp<0x114>(0u, v);
    v += dpp<0x118>(0u, v);
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x142, 0xa, 0xf, false));
    v += static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x143, 0xc, 0xf, false));
    return v;
}

}  // namespace irgs
