// MFMA 16x16x4 operand layout (one wave): lane l supplies A[i = l%16][k = l/16]
// and B[k = l/16][j = l%16].  Accumulator register r of lane l holds
// C[i][j = l%16] with i = 4*(l/16) + r for the f32 instruction and
// i = l/16 + 4*r for the f64 one (both measured on gfx950).
#pragma once

namespace sg {

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static __device__ inline acc_t run(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct Mfma<float> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static __device__ inline acc_t run(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

}  // namespace sg
