// bf16 pairs, operands of v_mfma_f32_16x16x32_bf16 and reductions over lanes, as the block and chunk kernels use them.
// Lane (r, g) = (lane % 16, lane / 16).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sla {
namespace lane_ops {

typedef __attribute__((ext_vector_type(4))) float f4;
typedef __attribute__((ext_vector_type(4))) uint32_t u4;
typedef __attribute__((ext_vector_type(2))) uint32_t u2;
typedef __attribute__((ext_vector_type(4))) short s4;
typedef __attribute__((ext_vector_type(8))) short s8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf8;
typedef __attribute__((address_space(3))) s4 lds_s4;

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ float bf_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float bf_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {  // the hardware conversion: nearest even, NaN kept
    bf2 t;
    t.x = (__bf16)lo;
    t.y = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, t);
}
__device__ __forceinline__ u2 pack4(f4 x) { return u2{pack2(x[0], x[1]), pack2(x[2], x[3])}; }
__device__ __forceinline__ s8 join(s4 a, s4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
// Lane (r, g) holds row r of A / column r of B, contraction slots of group g; D[4g + i][r] in register i.
__device__ __forceinline__ void mma(f4& c, s8 a, s8 b) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}
// Transposing LDS read: lane l of a group of 16 addresses row l / 4, piece l % 4 (four columns), and receives column
// l (element l % 4 of piece l / 4) of the four rows.
__device__ __forceinline__ s4 lds_tr(const uint16_t* p) { return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)p); }

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_all(float x) {  // sum over the 16 lanes of a row, to all
    x += dpp<0x128>(x);
    x += dpp<0x124>(x);
    x += dpp<0x122>(x);
    x += dpp<0x121>(x);
    return x;
}
// Sum over the four 16-lane rows of a wave, returned in every lane.
__device__ __forceinline__ float all_groups(float x) {
    const uint32_t xi = __float_as_uint(x);
    const u2 a = __builtin_amdgcn_permlane16_swap(xi, xi, false, false);
    const uint32_t yi = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    const u2 b = __builtin_amdgcn_permlane32_swap(yi, yi, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace lane_ops
}  // namespace sla
