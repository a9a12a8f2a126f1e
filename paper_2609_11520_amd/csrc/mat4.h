// Matrix-core products of complex blocks: the real and imaginary parts of 8 columns are the 16 columns of
// one real tile.
#pragma once
#include "common.h"

namespace fio {

// 16 x 16 tile of four reals per lane: lane l holds column l & 15
template <typename T> struct Mat4;
template <> struct Mat4<double> {
    using V = double __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mac(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return (lane >> 4) + 4 * i; }
};
template <> struct Mat4<float> {
    using V = float __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mac(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int i) { return 4 * (lane >> 4) + i; }
};

// the other half of a 16-lane row: lane l gets lane l xor 8
__device__ __forceinline__ float row_half(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));
}
__device__ __forceinline__ double row_half(double v) {
    const long b = __builtin_bit_cast(long, v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x128, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x128, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long)hi << 32) | (unsigned)lo);
}

}  // namespace fio
