// Device helpers shared by the HIP loop bodies (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jk {

constexpr int kWave = 64;

typedef double dvec2 __attribute__((ext_vector_type(2)));
// a pair at any 8-byte address (16-byte accesses need no more on this chip)
typedef double dpair __attribute__((ext_vector_type(2), aligned(8)));

// VEC consecutive doubles.
template <int VEC>
__device__ __forceinline__ void load_vec(const double *p, double (&v)[VEC]) {
    if constexpr (VEC == 2) {
        const dpair t = *reinterpret_cast<const dpair *>(p);
        v[0] = t.x;
        v[1] = t.y;
    } else {
        v[0] = *p;
    }
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Sum over each aligned group of G lanes by the butterfly xor 1, 2, 4, 8.  Once
// the lanes of a quad hold the same value, mirroring 8 lanes reaches the
// same value as xor 4 does, and mirroring 16 as xor 8.
template <int G>
__device__ __forceinline__ double group_sum(double s) {
    s += dpp<0xB1>(s);                          // quad_perm 1 0 3 2
    s += dpp<0x4E>(s);                          // quad_perm 2 3 0 1
    if constexpr (G >= 8) s += dpp<0x141>(s);   // row_half_mirror
    if constexpr (G >= 16) s += dpp<0x140>(s);  // row_mirror
    return s;
}

// Sum of `v` over the 64 lanes of a wave by a fixed butterfly (xor 1, 2, 4,
// ..., 32); every lane ends with the same value.
__device__ __forceinline__ double wave_sum(double v) {
    v = group_sum<16>(v);
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    return v;
}

// Workgroup sum in a fixed order: wave butterflies, then the wave results
// added in wave order by thread 0.  `sh` holds one double per wave.
__device__ __forceinline__ double block_sum(double v, double *sh) {
    const int tid = threadIdx.x + threadIdx.y * blockDim.x;
    const int nw = (blockDim.x * blockDim.y + kWave - 1) / kWave;
    v = wave_sum(v);
    if ((tid & (kWave - 1)) == 0) sh[tid / kWave] = v;
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
        for (int w = 0; w < nw; ++w) s += sh[w];
    return s;  // valid in thread 0
}

}  // namespace jk
