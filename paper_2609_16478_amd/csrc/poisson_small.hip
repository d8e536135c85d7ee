// Dirichlet solve on a small 2-D grid by one work-group (gfx950): w = L_int^{-1} g with the
// interior plane in LDS from the load of g to the store of w.
//
// As separate passes such a solve is five launches (seven where the tables are generated too)
// of a few microseconds of work each.  Here the four transforms run as half-size sine products
// on the matrix cores (see dst_direct.hip), from the plane in LDS through registers back to it;
// any lengths.  One work-group runs on one compute unit, so its own chain bounds it; FP64, one
// launch and separate passes (without a handle, with the tables' launches): 32^2 11 and 27 us,
// 64^2 (1.05e6 flops) 16 and 29 us, 80^2 (2.0e6) 30 and 28, 96^2 (3.5e6) 41 and 41; with a handle
// 64^2 19 and 24, 96^2 43 and 33.  POISSON_SMALL_FLOPS lies between 64^2 and 80^2.
#include "common.h"
#include "kernels.h"
#include "mfma_sine.h"

#include <algorithm>
#include <mutex>

namespace ahoc {

namespace {

constexpr int POISSON_UNITS = 2;  // units of 16 pencils x (16 odd + 16 even) outputs per wavefront
constexpr double POISSON_SMALL_FLOPS = 1.3e6;

// Row length of the plane in LDS: 2 (mod 32) FP64 or 4 (mod 64) FP32 entries, so that the 16
// rows of an operand read start 4 banks apart.
template <typename T> __host__ __device__ constexpr int plane_ld(int ni) {
  const int m = 256 / (int)sizeof(T), r = 16 / (int)sizeof(T);
  return (ni + m - 1 - r) / m * m + r;
}

// One transform of the plane x (rows of ld): the pencils are its rows (ROWS) or its columns.
// f(pencil, k, value) takes output k (from 0) of each pencil after every read of the plane.
template <typename T, bool ROWS, typename F>
__device__ __forceinline__ void plane_pass(const T* x, int ld, int N, int npencil, const T* tab, F&& f) {
  using S = SineOps<T>;
  using v4 = typename S::v4;
  const int L = N - 1, Hm = N / 2, two_n = 2 * N, pairs = (Hm + 15) / 16;
  const int units = (npencil + 15) / 16 * pairs, nw = blockDim.x >> 6, w = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  v4 ae[POISSON_UNITS], ao[POISSON_UNITS];
#pragma unroll
  for (int u = 0; u < POISSON_UNITS; ++u) {
    ae[u] = ao[u] = v4{T(0), T(0), T(0), T(0)};
    const int id = w + u * nw;
    if (id >= units) continue;
    const int p0 = id / pairs * 16, j0 = id % pairs * 16;
    const int p = min(p0 + li, npencil - 1);  // (past the last: another pencil's values, unused)
    const unsigned k = 2u * (j0 + li) + 1u;
    unsigned ie = (k % two_n) * (1u + lk) % two_n, io = ((k + 1u) % two_n) * (1u + lk) % two_n;
    const unsigned de = 4u * (k % two_n) % two_n, dd = 4u * ((k + 1u) % two_n) % two_n;
#pragma unroll 4
    for (int s = 0; s < Hm; s += 4) {
      const int m = 1 + s + lk;
      const int mc = min(m, Hm);
      T a = ROWS ? x[p * ld + mc - 1] : x[(mc - 1) * ld + p];
      T b = ROWS ? x[p * ld + N - mc - 1] : x[(N - mc - 1) * ld + p];
      if (m > Hm) a = T(0);
      if (m > Hm || 2 * m == N) b = T(0);
      const T be = a + b, bo = a - b, se = tab[sine_pad(ie)], so = tab[sine_pad(io)];
      ie += de;
      io += dd;
      ie = min(ie, ie - (unsigned)two_n);
      io = min(io, io - (unsigned)two_n);
      ae[u] = ROWS ? S::mfma(be, se, ae[u]) : S::mfma(se, be, ae[u]);
      ao[u] = ROWS ? S::mfma(bo, so, ao[u]) : S::mfma(so, bo, ao[u]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < POISSON_UNITS; ++u) {
    const int id = w + u * nw;
    if (id >= units) continue;
    const int p0 = id / pairs * 16, j0 = id % pairs * 16;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int p = p0 + (ROWS ? S::row(lk, r) : li), k = 2 * (j0 + (ROWS ? li : S::row(lk, r)));
      if (p >= npencil) continue;
      if (k < L) f(p, k, ae[u][r]);
      if (k + 1 < L) f(p, k + 1, ao[u][r]);
    }
  }
}

template <typename T> __global__ void __launch_bounds__(1024) k_poisson_small(PoissonSmall<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n0 = a.n[0], n1 = a.n[1], l0 = n0 - 1, l1 = n1 - 1;
  const int ld = plane_ld<T>(l0);
  T* x = reinterpret_cast<T*>(smem);
  T* tab0 = x + (size_t)l1 * ld;
  T* tab1 = tab0 + sine_pad(2 * n0);
  T* s0 = tab1 + sine_pad(2 * n1);
  T* s1 = s0 + l0;
  // period tables sin(pi j / N) and eigenvalues of both axes
  auto tables = [&](T* tab, T* s, int ax) {
    const int N = a.n[ax];
    const T* sn = a.sn[ax];
    for (int i = threadIdx.x; i < 2 * N; i += blockDim.x) {
      tab[sine_pad(i)] = sn ? sine_entry<T>(sn, N, a.half[ax], i) : (T)sinpi((double)i / N);
    }
    for (int i = threadIdx.x; i < N - 1; i += blockDim.x) {
      if (a.s[ax]) {
        s[i] = a.s[ax][i];
      } else {
        const double sv = sinpi((double)(i + 1) / (2.0 * N));
        s[i] = (T)(-4.0 * sv * sv / (a.h[ax] * a.h[ax]));
      }
    }
  };
  tables(tab0, s0, 0);
  tables(tab1, s1, 1);
  constexpr int U = 4;
  for (int e0 = threadIdx.x; e0 < l0 * l1; e0 += U * blockDim.x) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * blockDim.x;
      v[u] = a.g[min(e, l0 * l1 - 1)];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * blockDim.x;
      if (e < l0 * l1) x[e / l0 * ld + e % l0] = (T)v[u];
    }
  }
  __syncthreads();
  plane_pass<T, true>(x, ld, n0, l1, tab0, [&](int p, int k, T v) { x[p * ld + k] = v; });
  __syncthreads();
  plane_pass<T, false>(x, ld, n1, l0, tab1, [&](int p, int k, T v) {
    const T sa = s0[p];
    x[k * ld + p] = v * a.scale / (sa + (T(1) + a.c_ta * sa) * s1[k]);
  });
  __syncthreads();
  plane_pass<T, false>(x, ld, n1, l0, tab1, [&](int p, int k, T v) { x[k * ld + p] = v; });
  __syncthreads();
  plane_pass<T, true>(x, ld, n0, l1, tab0, [&](int p, int k, T v) { a.w[p * l0 + k] = (double)v; });
}

template <typename T> size_t small_lds(int n0, int n1) {
  return sizeof(T) *
         ((size_t)(n1 - 1) * plane_ld<T>(n0 - 1) + sine_pad(2 * n0) + sine_pad(2 * n1) + (n0 - 1) + (n1 - 1));
}
int small_units(int n0, int n1) {
  auto units = [](int N, int pencils) { return (pencils + 15) / 16 * ((N / 2 + 15) / 16); };
  return std::max(units(n0, n1 - 1), units(n1, n0 - 1));
}

template <typename T> bool small_fits(int n0, int n1) {
  return 2.0 * (dst_sine_flops(n0, n1 - 1, 1) + dst_sine_flops(n1, 1, n0 - 1)) <= POISSON_SMALL_FLOPS &&
         small_lds<T>(n0, n1) <= 160 * 1024 && small_units(n0, n1) <= 16 * POISSON_UNITS;
}

}  // namespace

template <typename T> bool poisson_small_ok(int n0, int n1) { return dst_get_variant() == 0 && small_fits<T>(n0, n1); }

template <typename T> int poisson_small(const PoissonSmall<T>& a, hipStream_t st) {
  const int n0 = a.n[0], n1 = a.n[1];
  if (n0 < 2 || n1 < 2 || !small_fits<T>(n0, n1)) return ST_UNSUPPORTED;
  const size_t lds = small_lds<T>(n0, n1);
  if (lds > 64 * 1024) {
    static std::once_flag once;
    std::call_once(once, [] {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_poisson_small<T>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
  }
  const int waves = std::max(4, std::min(16, small_units(n0, n1)));
  hipLaunchKernelGGL(k_poisson_small<T>, dim3(1), dim3(64 * waves), lds, st, a);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template bool poisson_small_ok<float>(int, int);
template bool poisson_small_ok<double>(int, int);
template int poisson_small<float>(const PoissonSmall<float>&, hipStream_t);
template int poisson_small<double>(const PoissonSmall<double>&, hipStream_t);

}  // namespace ahoc
