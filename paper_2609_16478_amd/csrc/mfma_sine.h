// Parts shared by the sine products on the matrix cores: the 16x16x4 product in the working
// precision, and the period table its sine operand is gathered from.
#pragma once

namespace ahoc {

template <typename T> struct SineOps;
template <> struct SineOps<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of the 16x16 result held in element r of lane group lk = lane / 16
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
  static constexpr int PAD = 4;  // LDS row padding of the row-pass tile -> conflict-free reads
};
template <> struct SineOps<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mfma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
  static constexpr int PAD = 2;
};

// Period table in LDS: one word of padding every 32, so that the strides 2 m of the 16 lanes'
// indices do not meet in one bank where m is a multiple of a power of two
__host__ __device__ constexpr int sine_pad(int j) { return j + (j >> 5); }

// sin(pi i / N), i = 0..2N-1, from the table of a length: a whole period, or (half) its quarter
// by sin(pi + t) = -sin t and sin(pi - t) = sin t.
template <typename T> __device__ __forceinline__ T sine_entry(const T* __restrict__ sn, int N, int half, int i) {
  const int j = i >= N ? i - N : i;
  const T v = sn[!half ? i : j > N / 2 ? N - j : j];
  return half && i >= N ? -v : v;
}

}  // namespace ahoc
