// FP32 products of small matrices with one column per lane, on the matrix
// cores (used by the 2-D and 3-D kernels).
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

namespace cmcg {

// FP32 products of small matrices with one column per lane on
// v_mfma_f32_4x4x1_16b_f32: with the A operand of one of the 16 blocks
// broadcast to all of them (cbsz = 4, abid = the block) an instruction adds
// A[4 g .. 4 g + 3][k] * column[k] to four rows of every lane's column, in the
// order and with the rounding of an fma() per row (checked on the GPU).  A
// register holds the operands of 16 instructions, so the matrices of an order
// take a few registers instead of LDS reads, four rows a time instead of one.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int NK, int G, typename F>
__device__ __forceinline__ void mfma_operand(float (&m)[(NK * G + 15) / 16], int lane, F at) {
#pragma unroll
    for (int v = 0; v < (NK * G + 15) / 16; ++v) {
        const int q = 16 * v + lane / 4;
        m[v] = q < NK * G ? at(4 * (q % G) + lane % 4, q / G) : 0.f;
    }
}
template <int NK, int G, int NX, size_t... I>
__device__ __forceinline__ void mfma_steps(const float (&m)[(NK * G + 15) / 16], const float (&x)[NX], f32x4 (&acc)[G],
                                           std::index_sequence<I...>) {
    ((acc[I % G] = __builtin_amdgcn_mfma_f32_4x4x1f32(m[I / 16], x[I / G], acc[I % G], 4, I % 16, 0)), ...);
}
template <int NK, int G, int NX>
__device__ __forceinline__ void mfma_rows(const float (&m)[(NK * G + 15) / 16], const float (&x)[NX], f32x4 (&acc)[G]) {
    static_assert(NX >= NK, "a column value per K step");
    mfma_steps<NK, G>(m, x, acc, std::make_index_sequence<NK * G>());
}
// One row group with K steps 0 .. NK/2 - 1 added to x0 and the rest to x1.
template <int NK, int NX, size_t... I>
__device__ __forceinline__ void mfma_pair_steps(const float (&m)[(NK + 15) / 16], const float (&x)[NX], f32x4& x0,
                                                f32x4& x1, std::index_sequence<I...>) {
    ((x0 = __builtin_amdgcn_mfma_f32_4x4x1f32(m[I / 16], x[I], x0, 4, I % 16, 0),
      x1 = __builtin_amdgcn_mfma_f32_4x4x1f32(m[(NK / 2 + I) / 16], x[NK / 2 + I], x1, 4, (NK / 2 + I) % 16, 0)),
     ...);
}
template <int NK, int NX>
__device__ __forceinline__ void mfma_pair(const float (&m)[(NK + 15) / 16], const float (&x)[NX], f32x4& x0, f32x4& x1) {
    static_assert(NK % 2 == 0 && NX >= NK, "two halves");
    mfma_pair_steps<NK>(m, x, x0, x1, std::make_index_sequence<NK / 2>());
}

}  // namespace cmcg
