// The boundary steps of one 2-D GMRES operator application on a square grid, one work-group
// per instance (gfx950).
//
// Between two Krylov vectors a step of w = S_h P^-1 v works on the four boundary lines alone
// until the V-solve's spectrum is generated, and again after the face sums: four transforms of
// lines of N - 1 values with pointwise work in between.  As separate passes these are seven
// launches whose work is a few microseconds each at most (six before the volume passes, two
// after them counting the gather).  Here the lines stay in LDS: opposite faces form the pencil
// pair of one complex FFT (dst_device.h), so that the preconditioner's 2 x 2 mode blocks act
// on the two components of one LDS entry, and the lift layers of both solves are read from the
// transformed lines' neighbours.  Latency bound: three transforms of one to four wavefronts in
// a row.
#include "dst_device.h"
#include "kernels.h"

#include <mutex>

namespace ahoc {

namespace fast {

namespace {

template <int N> using LPlan = PlanOf<N, N == 512 || N == 1024>;

// Positions of a pair in LDS from two global lines (len N - 1 each) and back.
template <typename T, int N, typename F> __device__ __forceinline__ void each_position(int t, F&& f) {
  constexpr int PPT = LPlan<N>::PPT, TPS = N / PPT;
#pragma unroll
  for (int k = 0; k < PPT; ++k) {
    const int m = 1 + t + k * TPS;
    if (k < PPT - 1 || m < N) f(m);
  }
}

// DST-I of the pair in seq (positions 1..N-1).
template <typename T, int N>
__device__ __forceinline__ void dst_pair(cx<T>* seq, cx<T>* tot, int t, const cx<T>* __restrict__ tw,
                                         const T* __restrict__ sn) {
  using PL = LPlan<N>;
  cx<T> A, B;
  A.x = A.y = T(1);
  B.x = B.y = T(0);
  pair_sync<N / PL::PPT>();
  pre_lds<T, N, PL>(seq, t, sn);
  fft<T, N, PL>(seq, t, tw);
  post<T, N, PL, false>(seq, tot, t, A, B, nullptr, T(0));
}

template <int N> constexpr int line_threads(int pairs) {
  return pairs * (N / LPlan<N>::PPT) < 64 ? 64 : pairs * (N / LPlan<N>::PPT);
}
template <typename T, int N> constexpr size_t front_lds() {
  return (2 * seq_stride<N>() + 4) * sizeof(cx<double>) + (4 * seq_stride<N>() + 8) * sizeof(cx<T>);
}

// z = P^-1 q (FP64; q itself without the preconditioner), in FP64 and, for an FP32 operator,
// converted; the lift layers of z for the V-solve (w0 across the face, wt to the neighbours
// along it) and of the U-solve (m1 z / alpha), transformed, in the layouts of face_lifts2.
template <typename T, int N>
__global__ void __launch_bounds__(line_threads<N>(4)) k_front2d(Front2d<T> a) {
  using PL = LPlan<N>;
  constexpr int TPS = N / PL::PPT, L = N - 1, LDQ = seq_stride<N>();
  static_assert(TPS <= 64 && 64 % TPS == 0, "a pair's lanes lie in one wavefront");
  extern __shared__ __align__(16) unsigned char smem[];
  cx<double>* sd = reinterpret_cast<cx<double>*>(smem);
  cx<double>* totd = sd + 2 * LDQ;
  cx<T>* st = reinterpret_cast<cx<T>*>(totd + 4);
  cx<T>* tott = st + 4 * LDQ;
  const long long b = blockIdx.x;
  const int p = threadIdx.x / TPS, t = threadIdx.x - p * TPS;
  if (p < 2) {  // pair 0: x-, x+; pair 1: y-, y+
    cx<double>* seq = sd + p * LDQ;
    const long long lo = b * 4 * L + 2 * p * L - 1, hi = lo + L;
    each_position<double, N>(t, [&](int m) {
      cx<double> v;
      v.x = a.q[lo + m];
      v.y = a.q[hi + m];
      seq[pad(m)] = v;
    });
    if (t == 0) seq[0] = cx<double>{0, 0};
    if (a.pc) {
      dst_pair<double, N>(seq, totd + 2 * p, t, a.twd, a.snd);
      const int ml = 2 * p * L - 1, mh = ml + L;
      each_position<double, N>(t, [&](int m) {
        const cx<double> v = seq[pad(m)];
        cx<double> o;
        o.x = a.pc[ml + m] * v.x + a.qc[ml + m] * v.y;
        o.y = a.qc[mh + m] * v.x + a.pc[mh + m] * v.y;
        seq[pad(m)] = o;
      });
      dst_pair<double, N>(seq, totd + 2 * p, t, a.twd, a.snd);
    }
    each_position<double, N>(t, [&](int m) {
      const cx<double> v = seq[pad(m)];
      if (a.z) {
        a.z[lo + m] = v.x;
        a.z[hi + m] = v.y;
      }
      if (a.zt) {
        a.zt[lo + m] = (T)v.x;
        a.zt[hi + m] = (T)v.y;
      }
    });
  }
  __syncthreads();
  if (p < 4) {  // pairs: V lift of the x faces, of the y faces, then the U-solve's
    const int ax = p & 1;
    const bool lift = p < 2;
    const cx<double>* z = sd + ax * LDQ;
    cx<T>* seq = st + p * LDQ;
    const T w0 = ax ? a.w0y : a.w0x;
    const T* ia = a.ia + b * a.nnodal;
    each_position<T, N>(t, [&](int m) {
      cx<T> o;
      const T zx = (T)z[pad(m)].x, zy = (T)z[pad(m)].y;
      if (lift) {
        o.x = w0 * zx + a.wt * (T)z[pad(m - 1)].x;
        o.y = w0 * zy + a.wt * (T)z[pad(m - 1)].y;
        if (m + 1 < N) {
          o.x += a.wt * (T)z[pad(m + 1)].x;
          o.y += a.wt * (T)z[pad(m + 1)].y;
        }
      } else {  // boundary nodes (0 | N, m) of the x faces, (m, 0 | N) of the y faces
        const long long n0 = ax ? m : (long long)m * (N + 1), n1 = ax ? (long long)N * (N + 1) + m : n0 + N;
        o.x = a.m1 * zx * ia[n0];
        o.y = a.m1 * zy * ia[n1];
      }
      seq[pad(m)] = o;
    });
    if (t == 0) seq[0] = cx<T>{0, 0};
    dst_pair<T, N>(seq, tott + 2 * p, t, a.tw, a.sn);
    const int len = ax ? a.px : L;
    T* out = (lift ? (ax ? a.Fy : a.Fx) : (ax ? a.Uy : a.Ux)) + b * 2 * len - 1;
    each_position<T, N>(t, [&](int m) {
      const cx<T> v = seq[pad(m)];
      out[m] = v.x;
      out[len + m] = v.y;
    });
  }
}

// y = af h^-2 S - z from the transformed face sums (Fx, Fy): the gather behind their transform.
template <typename T, int N>
__global__ void __launch_bounds__(line_threads<N>(2)) k_back2d(Back2d<T> a) {
  using PL = LPlan<N>;
  constexpr int TPS = N / PL::PPT, L = N - 1, LDQ = seq_stride<N>();
  extern __shared__ __align__(16) unsigned char smem[];
  cx<T>* st = reinterpret_cast<cx<T>*>(smem);
  cx<T>* tot = st + 2 * LDQ;
  const long long b = blockIdx.x;
  const int p = threadIdx.x / TPS, t = threadIdx.x - p * TPS;
  if (p >= 2) return;
  cx<T>* seq = st + p * LDQ;
  const int len = p ? a.px : L;
  const T* f = (p ? a.Fy : a.Fx) + b * 2 * len - 1;
  each_position<T, N>(t, [&](int m) {
    cx<T> v;
    v.x = f[m];
    v.y = f[len + m];
    seq[pad(m)] = v;
  });
  if (t == 0) seq[0] = cx<T>{0, 0};
  dst_pair<T, N>(seq, tot + 2 * p, t, a.tw, a.sn);
  const T ih2 = p ? a.ihy2 : a.ihx2;
  const long long lo = b * 4 * L + 2 * p * L - 1, hi = lo + L;
  each_position<T, N>(t, [&](int m) {
    const cx<T> v = seq[pad(m)];
    a.R[lo + m] = (double)(a.af[lo + m] * ih2 * v.x - a.z[lo + m]);
    a.R[hi + m] = (double)(a.af[hi + m] * ih2 * v.y - a.z[hi + m]);
  });
}

template <typename T, int N> int front_launch(const Front2d<T>& a, int nb, hipStream_t st) {
  constexpr size_t lds = front_lds<T, N>();
  static_assert(lds <= 160 * 1024, "");
  if (lds > 64 * 1024) {
    static std::once_flag once;
    std::call_once(once, [] {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_front2d<T, N>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
  }
  hipLaunchKernelGGL((k_front2d<T, N>), dim3(nb), dim3(line_threads<N>(4)), lds, st, a);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}
template <typename T, int N> int back_launch(const Back2d<T>& a, int nb, hipStream_t st) {
  constexpr size_t lds = (2 * seq_stride<N>() + 4) * sizeof(cx<T>);
  static_assert(lds <= 64 * 1024, "");
  hipLaunchKernelGGL((k_back2d<T, N>), dim3(nb), dim3(line_threads<N>(2)), lds, st, a);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

}  // namespace

}  // namespace fast

#define AHOC_LINES(F) F(32) F(64) F(96) F(128) F(192) F(256) F(384) F(512) F(768) F(1024)

bool lines2d_supported(int N) {
  switch (N) {
#define AHOC_L(NN) case NN:
    AHOC_LINES(AHOC_L)
#undef AHOC_L
    return true;
    default: return false;
  }
}
template <typename T> int front2d(int N, const Front2d<T>& a, int nb, hipStream_t st) {
  switch (N) {
#define AHOC_L(NN) case NN: return fast::front_launch<T, NN>(a, nb, st);
    AHOC_LINES(AHOC_L)
#undef AHOC_L
    default: return ST_UNSUPPORTED;
  }
}
template <typename T> int back2d(int N, const Back2d<T>& a, int nb, hipStream_t st) {
  switch (N) {
#define AHOC_L(NN) case NN: return fast::back_launch<T, NN>(a, nb, st);
    AHOC_LINES(AHOC_L)
#undef AHOC_L
    default: return ST_UNSUPPORTED;
  }
}
template int front2d<float>(int, const Front2d<float>&, int, hipStream_t);
template int front2d<double>(int, const Front2d<double>&, int, hipStream_t);
template int back2d<float>(int, const Back2d<float>&, int, hipStream_t);
template int back2d<double>(int, const Back2d<double>&, int, hipStream_t);

}  // namespace ahoc
