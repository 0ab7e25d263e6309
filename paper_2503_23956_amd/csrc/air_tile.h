// MFMA operands and the layouts of the compacted cache, for both storage types and head sizes.
//
// Every matrix product of the library has 16 x 16 output tiles.  A lane (n = lane % 16, c = lane / 16) supplies 16 bytes
// of an operand at a time: of row (or column) n, the c-th quarter of a slice of kSlice contraction indices:
//   bf16  8 elements a lane, slices of 32: one v_mfma_f32_16x16x32_bf16
//   fp32  4 elements a lane, slices of 16: four v_mfma_f32_16x16x4_f32 (element i of every lane's 16 bytes in product i;
//         the order of the contraction indices is the lanes' own, the same for both operands), full fp32 products and sums.
//         256 flop a clock and CU: with 16 rows per key 512 bytes long that is 77 GB/s a CU for both products of decode,
//         2.5 times the 31 GB/s a CU gets of HBM when all of them stream.
#pragma once

#include "air_device.h"

namespace air {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

template <typename T>
struct Elem;
template <>
struct Elem<bf16_t> {
    static constexpr int kVec = 8;     // elements in 16 bytes
    static constexpr int kSlice = 32;  // contraction indices of one operand load
    static constexpr int kVTok = 32;   // tokens of a V' block
};
template <>
struct Elem<float> {
    static constexpr int kVec = 4, kSlice = 16, kVTok = 16;
};

template <typename T>
__device__ __forceinline__ f32x4 mma(const uint4 &a, const uint4 &b, f32x4 acc);
template <>
__device__ __forceinline__ f32x4 mma<bf16_t>(const uint4 &a, const uint4 &b, f32x4 acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ f32x4 mma<float>(const uint4 &a, const uint4 &b, f32x4 acc) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], acc, 0, 0, 0);
    return acc;
}

// products of the elements of two 16-byte pieces, added to sum in order
template <typename T>
__device__ __forceinline__ float dot_piece(const uint4 &a, const uint4 &b, float sum);
template <>
__device__ __forceinline__ float dot_piece<bf16_t>(const uint4 &a, const uint4 &b, float sum) {
    const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        sum = fmaf(__uint_as_float(x[w] << 16), __uint_as_float(y[w] << 16), sum);
        sum = fmaf(__uint_as_float(x[w] & 0xffff0000u), __uint_as_float(y[w] & 0xffff0000u), sum);
    }
    return sum;
}
template <>
__device__ __forceinline__ float dot_piece<float>(const uint4 &a, const uint4 &b, float sum) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int w = 0; w < 4; ++w) sum = fmaf(x[w], y[w], sum);
    return sum;
}

}  // namespace air
