// DST-I pass for transform lengths without a radix-2/3 FFT plan (gfx950).
//
// X_k = sum_{m=1}^{N-1} x_m sin(pi k m / N), k = 1..N-1, O(N) work per output, with
// sin(pi j / N) read from a one-period table (index k m mod 2N, advanced incrementally).
// It gives every grid length from the one-sided formula's minimum (N_a >= 4, Sec. 2.2)
// upward a pass with the same layouts as the FFT kernels: rows (contiguous pencils, `pitch`
// apart) or strided pencils [outer][L][inner].  The fused form (slowest axis of a Poisson
// solve) transforms, multiplies mode k of column c by scale / (A_c + B_c s_this[k-1]) -- the
// compact Laplacian's eigenvalue, Sec. 2.3 -- and transforms back.
//
// k_dst_sine runs the sums on the matrix cores as two half-size products: with
// sin(pi k (N-m) / N) = (-1)^(k+1) sin(pi k m / N), odd outputs are sums over m <= N/2 of
// e_m = x_m + x_{N-m}, even ones of o_m = x_m - x_{N-m} (e = x_m at m = N/2), N^2 flops per
// pencil, accumulated in the working precision.  What bounds it: the matrix cores from N of
// about 200 (FP64, 128 flop per cycle and CU) upward, memory below.  A wavefront owns TO pairs
// of 16 odd and 16 even outputs next to each other for TP x 16 pencils; e and o of a chunk of m
// are staged in LDS once for all of them.  The sine operand is gathered from the period table
// in LDS instead of read as a stored matrix: no N^2 / 2 table per length (16 MB at N = 2000)
// that each handle would build and each work-group stream through L2, and the gather's bank
// conflicts hide behind the MFMAs (64 cycles each in FP64) once two pencil tiles share it.
// Against one thread per output (the form this replaces): FP32 along y of 199 x 149 x 119
// points 549 -> 19 us a call, an FP64 Poisson solve of 99 x 89 x 74 points 227 -> 61 us, a 2-D
// 500 x 300 FP64 solve (25 GMRES iterations) 118.8 -> 7.4 ms (3.5 with the Krylov step and
// the faces in few launches); errors against 64-bit sums no larger (FP32 2.2e-7 -> 1.6e-7).  Where a pass has few pencils (lines of 2-D faces) its time
// is latency: four lines of N = 1024 in FP64 took 25 us with a 128-step sum per wavefront and
// staging loops that waited for each load, 10.7 us with the sum split over four wavefronts and
// one trip to memory.
// k_dst_direct, one thread per output and the whole pencil in LDS, remains for in-place
// passes of N > 2048, whose outputs k_dst_sine could not hold in registers, and for short strided
// pencils (see short_pencils).
#include "common.h"
#include "mfma_sine.h"

#include <algorithm>
#include <mutex>

namespace ahoc {

namespace {

template <typename T> struct DirectArgs {
  const T* in;
  T* out;
  const T* sn2;       // sin(pi j / N), j = 0..2N-1
  int N;
  int P;              // pencils per work-group
  long long outer, inner, pitch;
  long long ntile_inner;
  int cols;
  bool fused;
  DstScale<T> fs;
};

// y_k = sum_m x_m sin(pi k m / N) for k = 1..L over the pencils of the tile held in `x`
// (pencil p at x + p * L), into y (same layout); threads take (p, k) with k fastest.
template <typename T>
__device__ void direct_sums(const T* x, T* y, int P, int L, int N, const T* __restrict__ sn2) {
  const int two_n = 2 * N;
  for (int e = threadIdx.x; e < P * L; e += blockDim.x) {
    const int p = e / L;
    const int k = e - p * L + 1;
    const T* xp = x + (long long)p * L;
    T acc = 0;
    int idx = 0;
    for (int m = 1; m <= L; ++m) {
      idx += k;
      if (idx >= two_n) idx -= two_n;
      acc += xp[m - 1] * sn2[idx];
    }
    y[e] = acc;
  }
}

template <typename T> __global__ void __launch_bounds__(256) k_dst_direct(DirectArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  T* x = reinterpret_cast<T*>(smem);
  const int L = a.N - 1;
  const int P = a.P;
  T* y = x + (long long)P * L;
  const bool rows = a.inner == 1;
  long long base, c0 = 0;
  int ncols;
  if (rows) {
    base = (long long)blockIdx.x * P;
    const long long left = a.outer - base;
    ncols = left < P ? (int)left : P;
  } else {
    const long long o = blockIdx.x / a.ntile_inner;
    c0 = (blockIdx.x - o * a.ntile_inner) * (long long)P;
    base = o * (long long)L * a.inner + c0;
    const long long left = a.inner - c0;
    ncols = left < P ? (int)left : P;
  }
  // load: rows with m fastest, strided pencils with the column fastest (coalesced)
  for (int e = threadIdx.x; e < P * L; e += blockDim.x) {
    int p, m;
    if (rows) {
      p = e / L;
      m = e - p * L;
    } else {
      m = e / P;
      p = e - m * P;
    }
    T v = 0;
    if (p < ncols) v = rows ? a.in[(base + p) * a.pitch + m] : a.in[base + (long long)m * a.inner + p];
    x[p * L + m] = v;
  }
  __syncthreads();
  T* res = y;
  if (a.fused) {
    direct_sums<T>(x, y, P, L, a.N, a.sn2);
    __syncthreads();
    for (int e = threadIdx.x; e < P * L; e += blockDim.x) {
      const int p = e / L;
      const int k = e - p * L + 1;
      const long long col = c0 + p;
      const long long ib = col / a.fs.na;
      const long long ia = col - ib * a.fs.na;
      T A = 1, B = 0;
      if (col < a.inner && ia < a.fs.nva) {
        const T sa = a.fs.s_a[ia];
        const T sb = a.fs.s_b ? a.fs.s_b[ib] : T(0);
        A = sa + sb + a.fs.c_ab * sa * sb + a.fs.a0 + a.fs.ka * sa + a.fs.kb * sb;
        B = T(1) + a.fs.c_ta * sa + a.fs.c_tb * sb + a.fs.kt;
      }
      y[e] *= a.fs.scale / (A + B * a.fs.s_this[k - 1]);
    }
    __syncthreads();
    direct_sums<T>(y, x, P, L, a.N, a.sn2);
    __syncthreads();
    res = x;
  } else {
    direct_sums<T>(x, y, P, L, a.N, a.sn2);
    __syncthreads();
  }
  for (int e = threadIdx.x; e < P * L; e += blockDim.x) {
    int p, k;
    if (rows) {
      p = e / L;
      k = e - p * L;
    } else {
      k = e / P;
      p = e - k * P;
    }
    if (p >= ncols) continue;
    const T v = res[p * L + k];
    if (rows) a.out[(base + p) * a.pitch + k] = v;
    else a.out[base + (long long)k * a.inner + p] = v;
  }
  if (rows)
    for (int e = threadIdx.x; e < ncols * (a.cols - L); e += blockDim.x) {
      const int p = e / (a.cols - L);
      a.out[(base + p) * a.pitch + L + (e - p * (a.cols - L))] = T(0);
    }
}

template <typename T> struct SineArgs {
  const T* in;
  T* out;
  const T* sn;        // sin(pi j / N): j = 0..2N-1, or (half, even N) j = 0..N/2
  int N;
  int half;
  int cols;           // columns stored per row: L, or more (zeros) up to the row's pitch
  long long outer, inner, pitch;
  long long ntile_inner;
};

// Words of one half's (e or o) tile of mc values of m (a multiple of 64: conflict-free rows)
template <typename T, bool ROWS, int TP> constexpr int sine_half(int mc) {
  return ROWS ? 16 * TP * (mc + SineOps<T>::PAD) : mc * (TP == 1 ? 16 : 16 * TP + 16);
}
// lambda = A + B s_this of column `col`
template <typename T> __device__ __forceinline__ void sine_lambda(const DstScale<T>& fs, long long col, bool in, T* A, T* B) {
  const long long ib = col / fs.na;
  const long long ia = col - ib * fs.na;
  *A = 1;
  *B = 0;
  if (in && ia < fs.nva) {
    const T sa = fs.s_a[ia];
    const T sb = fs.s_b ? fs.s_b[ib] : T(0);
    *A = sa + sb + fs.c_ab * sa * sb + fs.a0 + fs.ka * sa + fs.kb * sb;
    *B = T(1) + fs.c_ta * sa + fs.c_tb * sb + fs.kt;
  }
}

// The outputs of TO pairs per KS wavefronts, from pair `first` on, of tile `tile` of 16 TP
// pencils.  KS wavefronts take every KS-th step of the sum over m and add their sums up at the
// end (in wavefront order): where a pass has so few pencils that most of the chip is idle, its
// time is the length of that chain.  mc: values of m staged at a time.
// In place (one work-group holds every output of the tile) the tile's reads end, at a barrier,
// before its writes.  scaled (strided pencils): eigen scaling by fs before the store.
template <typename T, bool ROWS, int TO, int TP, int KS>
__device__ __forceinline__ void sine_tile(const SineArgs<T>& a, const DstScale<T>& fs, bool scaled, long long tile,
                                          int first, bool in_place, int mc) {
  using S = SineOps<T>;
  using v4 = typename S::v4;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int P = 16 * TP;
  const int LDX = mc + S::PAD;                 // rows: [pencil][m]
  constexpr int LDC = TP == 1 ? 16 : P + 16;   // strided: [m][pencil]
  T* xe = reinterpret_cast<T*>(smem);
  T* xo = xe + sine_half<T, ROWS, TP>(mc);
  T* tab = xo + sine_half<T, ROWS, TP>(mc);
  const int N = a.N, L = N - 1, two_n = 2 * N, Hm = N / 2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nt = blockDim.x;
  const int li = lane & 15, lk = lane >> 4;
  long long base, c0 = 0;
  int ncols;
  if (ROWS) {
    base = tile * P;
    const long long left = a.outer - base;
    ncols = left < P ? (int)left : P;
  } else {
    const long long o = tile / a.ntile_inner;
    c0 = (tile - o * a.ntile_inner) * (long long)P;
    base = o * (long long)L * a.inner + c0;
    const long long left = a.inner - c0;
    ncols = left < P ? (int)left : P;
  }
  // Period table.  The kernels of few accumulators have up to TU entries per thread in flight
  // with the first tile loads and put them into LDS after those (11.9 -> 11.5 us a pass of
  // 300 x 499, FP64: one wait on memory instead of two); the others have no registers for them.
  constexpr bool early = TO * TP <= 2;
  constexpr int TU = early ? 4 : 1;
  auto entry = [&](int i) { return sine_entry<T>(a.sn, N, a.half, i); };
  T tv[TU];
  if constexpr (early) {
#pragma unroll
    for (int u = 0; u < TU; ++u) tv[u] = entry(min((int)threadIdx.x + u * nt, two_n - 1));
  } else {
    for (int i = threadIdx.x; i < two_n; i += nt) tab[sine_pad(i)] = entry(i);
  }
  bool pending = early;
  auto table = [&]() {
    pending = false;
#pragma unroll
    for (int u = 0; u < TU; ++u) {
      const int i = threadIdx.x + u * nt;
      if (i < two_n) tab[sine_pad(i)] = tv[u];
    }
    for (int i = threadIdx.x + TU * nt; i < two_n; i += nt) tab[sine_pad(i)] = entry(i);
  };
  // this lane's outputs of pair t: k = 2 j + 1 (odd) and 2 j + 2 (even), j = j0[t] + li; its
  // sine index starts at m = 1 + lk (the wavefront's first step) and advances by 4 KS k per
  // step, modulo the period
  const int wk = KS > 1 ? w % KS : 0;
  const int p0 = first + w / KS * TO;
  unsigned ie[TO], io[TO], de[TO], dd[TO];
#pragma unroll
  for (int t = 0; t < TO; ++t) {
    const unsigned k = 2u * (16u * (p0 + t) + li) + 1u;
    ie[t] = (k % two_n) * (1u + lk + 4u * wk) % two_n;
    io[t] = ((k + 1u) % two_n) * (1u + lk + 4u * wk) % two_n;
    de[t] = 4u * KS * (k % two_n) % two_n;
    dd[t] = 4u * KS * ((k + 1u) % two_n) % two_n;
  }
  v4 ae[TO][TP], ao[TO][TP];
#pragma unroll
  for (int t = 0; t < TO; ++t)
#pragma unroll
    for (int b = 0; b < TP; ++b) ae[t][b] = ao[t][b] = v4{T(0), T(0), T(0), T(0)};
  for (int m0 = 0; m0 < Hm; m0 += mc) {
    const int kc = Hm - m0 < mc ? (Hm - m0 + 3) & ~3 : mc;
    if (m0) __syncthreads();  // the last chunk's reads are done
    // eight positions per thread and step, their sixteen loads in flight together (four in the
    // FP64 row passes of up to 1024 threads, whose registers hold no more)
    constexpr int U = ROWS && sizeof(T) == 8 && KS == 1 ? 4 : 8;
    // (rows past the last are left as they are: a pencil's sums read only its own tile entries)
    const int todo = kc * (ROWS ? ncols : P);
    for (int e0 = threadIdx.x; e0 < todo; e0 += U * nt) {
      T x[U], y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * nt;
        const int p = ROWS ? e / kc : e % P, q = ROWS ? e - p * kc : e / P;
        const int m = m0 + q + 1;
        const bool ok = e < todo && m <= Hm && p < ncols;
        const T* src = ROWS ? a.in + (base + p) * a.pitch : a.in + base + p;
        const long long st = ROWS ? 1 : a.inner;
        x[u] = ok ? src[(m - 1) * st] : T(0);
        y[u] = ok && 2 * m != N ? src[(N - m - 1) * st] : T(0);
      }
      if (pending) table();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * nt;
        const int p = ROWS ? e / kc : e % P, q = ROWS ? e - p * kc : e / P;
        if (e < todo) {
          const int at = ROWS ? p * LDX + q : q * LDC + p;
          xe[at] = x[u] + y[u];
          xo[at] = x[u] - y[u];
        }
      }
    }
    if (pending) table();
    __syncthreads();
#pragma unroll 4
    for (int s = 4 * wk; s < kc; s += 4 * KS) {
      T be[TP], bo[TP];
#pragma unroll
      for (int b = 0; b < TP; ++b) {
        const int at = ROWS ? (16 * b + li) * LDX + s + lk : (s + lk) * LDC + 16 * b + li;
        be[b] = xe[at];
        bo[b] = xo[at];
      }
#pragma unroll
      for (int t = 0; t < TO; ++t) {
        const T se = tab[sine_pad(ie[t])], so = tab[sine_pad(io[t])];
        ie[t] += de[t];
        io[t] += dd[t];
        ie[t] = min(ie[t], ie[t] - (unsigned)two_n);
        io[t] = min(io[t], io[t] - (unsigned)two_n);
#pragma unroll
        for (int b = 0; b < TP; ++b) {
          if (ROWS) {
            ae[t][b] = S::mfma(be[b], se, ae[t][b]);
            ao[t][b] = S::mfma(bo[b], so, ao[t][b]);
          } else {
            ae[t][b] = S::mfma(se, be[b], ae[t][b]);
            ao[t][b] = S::mfma(so, bo[b], ao[t][b]);
          }
        }
      }
    }
  }
  if (in_place) __syncthreads();
  if constexpr (KS > 1) {
    // [output group][wavefront][value][lane] over the tile's LDS
    constexpr int NV = TO * TP * 8;
    __syncthreads();
    T* red = xe + (w / KS) * (KS - 1) * NV * 64;
#pragma unroll
    for (int t = 0; t < TO; ++t)
#pragma unroll
      for (int b = 0; b < TP; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (wk) {
            red[((wk - 1) * NV + (t * TP + b) * 8 + r) * 64 + lane] = ae[t][b][r];
            red[((wk - 1) * NV + (t * TP + b) * 8 + 4 + r) * 64 + lane] = ao[t][b][r];
          }
    __syncthreads();
    if (wk) return;
#pragma unroll
    for (int k = 0; k < KS - 1; ++k)
#pragma unroll
      for (int t = 0; t < TO; ++t)
#pragma unroll
        for (int b = 0; b < TP; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            ae[t][b][r] += red[(k * NV + (t * TP + b) * 8 + r) * 64 + lane];
            ao[t][b][r] += red[(k * NV + (t * TP + b) * 8 + 4 + r) * 64 + lane];
          }
  }
#pragma unroll
  for (int b = 0; b < TP; ++b) {
    T A = 1, B = 0, sc = 1;
    if (!ROWS && scaled) {
      const long long col = c0 + 16 * b + li;
      sc = fs.scale;
      sine_lambda<T>(fs, col, col < a.inner, &A, &B);
    }
#pragma unroll
    for (int t = 0; t < TO; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int p = 16 * b + (ROWS ? S::row(lk, r) : li);
        const int k = 2 * (16 * (p0 + t) + (ROWS ? li : S::row(lk, r)));  // positions k, k + 1 (from 0)
        if (p >= ncols) continue;
        T ve = ae[t][b][r], vo = ao[t][b][r];
        if (!ROWS && scaled) {
          if (k < L) ve *= sc / (A + B * fs.s_this[k]);
          if (k + 1 < L) vo *= sc / (A + B * fs.s_this[k + 1]);
        }
        T* op = ROWS ? a.out + (base + p) * a.pitch + k : a.out + base + (long long)k * a.inner + p;
        if (k < (ROWS ? a.cols : L)) op[0] = k < L ? ve : T(0);
        if (k + 1 < (ROWS ? a.cols : L)) op[ROWS ? 1 : a.inner] = k + 1 < L ? vo : T(0);
      }
    }
  }
}

// The same for N <= SINE_CHAIN_N, one pair of 16 odd and 16 even outputs of 16 pencils per
// work-group: each of the four wavefronts has its quarter of the sum, C steps of four m, straight
// from memory in registers, all in flight with the period table, and no tile to stage and wait
// for.  The faces of 128^3, 6 passes in a launch: 6.6 -> 5.0 us in FP64, 6.2 -> 5.2 in FP32.  From
// N of about 300 the rows' 32-byte pieces cost more than the staging: 500 x 300 points in FP64
// 13.6 us against 11.5 along x, 9.2 against 9.1 along y.
constexpr int SINE_CHAIN_N = 256;
template <typename T, bool ROWS, int C>
__device__ __forceinline__ void sine_chain(const SineArgs<T>& a, const DstScale<T>& fs, bool scaled, long long tile,
                                           int pair) {
  using S = SineOps<T>;
  using v4 = typename S::v4;
  extern __shared__ __align__(16) unsigned char smem[];
  T* red = reinterpret_cast<T*>(smem);  // [wavefront][value][lane]
  T* tab = red + 4 * 8 * 64;
  const int N = a.N, L = N - 1, Hm = N / 2, two_n = 2 * N;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  long long base, c0 = 0;
  int ncols;
  if (ROWS) {
    base = tile * 16 * a.pitch;
    ncols = (int)min(16LL, a.outer - tile * 16);
  } else {
    const long long o = tile / a.ntile_inner;
    c0 = (tile - o * a.ntile_inner) * 16;
    base = o * (long long)L * a.inner + c0;
    ncols = (int)min(16LL, a.inner - c0);
  }
  constexpr int TU = C / 4;  // 2 N <= 256 TU
  T tv[TU];
#pragma unroll
  for (int u = 0; u < TU; ++u) tv[u] = sine_entry<T>(a.sn, N, a.half, min((int)threadIdx.x + u * 256, two_n - 1));
  const int quarter = (Hm + 15) / 16 * 4, m0 = w * quarter;  // this wavefront's m: m0 + 1 ..
  // bytes within the tile's slab or rows (below 4 GiB: the rule of the dispatch)
  const unsigned sm = (ROWS ? 1u : (unsigned)a.inner) * sizeof(T);
  const unsigned sp = (unsigned)min(li, ncols - 1) * (ROWS ? (unsigned)a.pitch * (unsigned)sizeof(T) : (unsigned)sizeof(T));
  const char* src = reinterpret_cast<const char*>(a.in + base);
  auto at = [&](int row) { return *reinterpret_cast<const T*>(src + (row * sm + sp)); };
  unsigned k = 32u * pair + 2u * li + 1u;
  const unsigned ke = (int)k < N ? k : 0u, ko = (int)k + 1 < N ? k + 1u : 0u;
  unsigned ie = ke * (unsigned)(m0 + 1 + lk) % two_n, io = ko * (unsigned)(m0 + 1 + lk) % two_n;
  const unsigned de = 4u * ke % two_n, dd = 4u * ko % two_n;
  v4 ae = v4{T(0), T(0), T(0), T(0)}, ao = ae;
  for (int s0 = 0; s0 < quarter; s0 += 4 * C) {
    T x[C], y[C];
#pragma unroll
    for (int s = 0; s < C; ++s) {
      const int m = min(m0 + s0 + 4 * s + lk + 1, Hm);
      x[s] = at(m - 1);
      y[s] = at(N - m - 1);
    }
    if (s0 == 0) {
#pragma unroll
      for (int u = 0; u < TU; ++u) {
        const int i = threadIdx.x + u * 256;
        if (i < two_n) tab[sine_pad(i)] = tv[u];
      }
      __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < C; ++s) {
      const int q = s0 + 4 * s, m = m0 + q + lk + 1;
      const bool ok = q < quarter && m <= Hm;
      const T vs = 2 * m == N ? T(0) : y[s];
      const T e = ok ? x[s] + vs : T(0), o = ok ? x[s] - vs : T(0);
      const T se = tab[sine_pad(ie)], so = tab[sine_pad(io)];
      ie = min(ie + de, ie + de - two_n);
      io = min(io + dd, io + dd - two_n);
      ae = ROWS ? S::mfma(e, se, ae) : S::mfma(se, e, ae);
      ao = ROWS ? S::mfma(o, so, ao) : S::mfma(so, o, ao);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    red[(w * 8 + r) * 64 + lane] = ae[r];
    red[(w * 8 + 4 + r) * 64 + lane] = ao[r];
  }
  __syncthreads();
  // wavefront w adds up and stores the results' element w
  T ve = red[w * 64 + lane], vo = red[(4 + w) * 64 + lane];
#pragma unroll
  for (int q = 1; q < 4; ++q) {
    ve += red[(q * 8 + w) * 64 + lane];
    vo += red[(q * 8 + 4 + w) * 64 + lane];
  }
  const int p = ROWS ? S::row(lk, w) : li, kk = 32 * pair + 2 * (ROWS ? li : S::row(lk, w));  // positions kk, kk + 1
  if (p >= ncols) return;
  if (!ROWS && scaled) {
    T A, B;
    sine_lambda<T>(fs, c0 + li, true, &A, &B);
    if (kk < L) ve *= fs.scale / (A + B * fs.s_this[kk]);
    if (kk + 1 < L) vo *= fs.scale / (A + B * fs.s_this[kk + 1]);
  }
  T* op = a.out + base + (ROWS ? p * a.pitch + kk : (long long)kk * a.inner + p);
  if (kk < (ROWS ? a.cols : L)) op[0] = kk < L ? ve : T(0);
  if (kk + 1 < (ROWS ? a.cols : L)) op[ROWS ? 1 : a.inner] = kk + 1 < L ? vo : T(0);
}

// grid.x: tiles; grid.y: groups of blockDim.x / 64 / KS * TO output pairs (one group in place)
template <typename T, bool ROWS, int TO, int TP, int KS>
__global__ void __launch_bounds__(KS > 1 ? 256 : 1024) k_dst_sine(SineArgs<T> a, DstScale<T> fs, int scaled, int mc) {
  sine_tile<T, ROWS, TO, TP, KS>(a, fs, scaled != 0, blockIdx.x, blockIdx.y * ((blockDim.x >> 6) / KS) * TO,
                                 gridDim.y == 1, mc);
}

// grid.x: tiles; grid.y: output pairs
template <typename T, bool ROWS, int C>
__global__ void __launch_bounds__(256) k_dst_sine_chain(SineArgs<T> a, DstScale<T> fs, int scaled) {
  sine_chain<T, ROWS, C>(a, fs, scaled != 0, blockIdx.x, blockIdx.y);
}

// Several passes in one launch (the faces of a grid: a few thousand pencils in up to six
// arrays, whose separate launches each cost more than their work).  Work-groups of four
// wavefronts, 128 / KS outputs of 16 pencils each (CHAIN: its steps in flight, else 0).
constexpr int SINE_JOBS_MAX = 6;
template <typename T> struct SineJobs {
  SineArgs<T> job[SINE_JOBS_MAX];
  int end[SINE_JOBS_MAX];     // end of the job's work-groups
  int groups[SINE_JOBS_MAX];  // output groups of a tile
  int mc;
};
template <typename T, bool ROWS, int KS, int CHAIN>
__global__ void __launch_bounds__(256) k_dst_sine_jobs(SineJobs<T> s) {
  int j = 0;
  while ((int)blockIdx.x >= s.end[j]) ++j;
  const int b = (int)blockIdx.x - (j ? s.end[j - 1] : 0), g = s.groups[j];
  if constexpr (CHAIN) sine_chain<T, ROWS, CHAIN>(s.job[j], DstScale<T>(), false, b / g, b % g);
  else sine_tile<T, ROWS, 1, 1, KS>(s.job[j], DstScale<T>(), false, b / g, b % g * (4 / KS), false, s.mc);
}

constexpr size_t DIRECT_LDS_MAX = 160 * 1024;
constexpr long long SINE_CHAIN_WGS = 256;  // fewer work-groups than this: the sums over m are split too

template <typename T> void set_direct_lds_attr() {
  static std::once_flag once;
  std::call_once(once, [] {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dst_direct<T>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)DIRECT_LDS_MAX);
  });
}

template <typename K> int sine_lds(K* kernel, size_t lds, std::once_flag& once) {
  if (lds > DIRECT_LDS_MAX) return ST_UNSUPPORTED;
  if (lds > 64 * 1024)
    std::call_once(once, [&] {
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)DIRECT_LDS_MAX);
    });
  return ST_OK;
}
template <typename T, bool ROWS, int TP> size_t sine_lds_bytes(int N, int mc) {
  return sizeof(T) * (2 * (size_t)sine_half<T, ROWS, TP>(mc) + sine_pad(2 * N));
}
// m values staged at a time: 2048 / P for the passes that fill the chip (32 KB of FP64, several
// work-groups per CU); where one chain is the time, as many as there are up to 512 (one trip to
// memory).
int sine_mc(int N, int P, bool chain) {
  const int full = chain ? 512 : 2048 / P;
  int mc = 64;
  while (mc < full && mc < N / 2) mc *= 2;
  return mc;
}

template <typename T> size_t sine_chain_lds(int N) { return sizeof(T) * (4 * 8 * 64 + (size_t)sine_pad(2 * N)); }
// Offsets within 16 rows stay below 4 GiB
template <typename T> bool sine_chain_ok(const SineArgs<T>& a, bool rows) {
  return a.N <= SINE_CHAIN_N && (!rows || a.pitch < (1 << 24)) && (rows || a.inner < (1 << 18));
}

template <typename T, bool ROWS, int TO, int TP, int KS = 1>
int sine_launch(const SineArgs<T>& a, const DstScale<T>* fs, long long tiles, int groups, int waves, hipStream_t st) {
  if (tiles > 0x7fffffffLL || groups > 65535) return ST_UNSUPPORTED;
  const int mc = sine_mc(a.N, 16 * TP, KS > 1);
  const size_t lds = sine_lds_bytes<T, ROWS, TP>(a.N, mc);
  static std::once_flag once;
  TRY_ST(sine_lds(&k_dst_sine<T, ROWS, TO, TP, KS>, lds, once));
  hipLaunchKernelGGL((k_dst_sine<T, ROWS, TO, TP, KS>), dim3((unsigned)tiles, (unsigned)groups), dim3(64 * waves),
                     lds, st, a, fs ? *fs : DstScale<T>(), fs ? 1 : 0, mc);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename T, bool ROWS>
int sine_chain_launch(const SineArgs<T>& a, const DstScale<T>* fs, long long tiles, int pairs, hipStream_t st) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles, (unsigned)pairs), dim3(256), sine_chain_lds<T>(a.N), st, a,
                       fs ? *fs : DstScale<T>(), fs ? 1 : 0);
  };
  if (a.N <= 128) launch(k_dst_sine_chain<T, ROWS, 4>);
  else launch(k_dst_sine_chain<T, ROWS, 8>);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

// Whether a pass of `tiles` 16-pencil tiles that writes elsewhere than it reads splits its outputs
// over work-groups of four wavefronts (each re-reads the tile): while whole pencils would give
// fewer than two work-groups per CU, and their sums over the four wavefronts too while even those
// would leave compute units idle (SINE_CHAIN_WGS); and where a tile's outputs exceed one
// work-group's registers.
bool sine_splits(int N, long long tiles) {
  const int pairs = (N / 2 + 15) / 16;
  return pairs > 64 || (pairs > 1 && tiles < 512 && (pairs > 4 || tiles * ((pairs + 3) / 4) < SINE_CHAIN_WGS));
}

// Tiles of 32 pencils share each gathered sine between two MFMAs, 16-pencil tiles double the
// work-groups: 32 from two work-groups per CU upward.
template <typename T, bool ROWS>
int sine_pass(SineArgs<T>& a, const DstScale<T>* fs, bool disjoint, hipStream_t st) {
  const int pairs = (a.N / 2 + 15) / 16;
  auto tiles = [&](int P) {
    a.ntile_inner = ROWS ? 1 : (a.inner + P - 1) / P;
    return ROWS ? (a.outer + P - 1) / P : a.outer * a.ntile_inner;
  };
  if (disjoint && pairs > 64) return sine_launch<T, ROWS, 2, 2>(a, fs, tiles(32), (pairs + 15) / 16, 8, st);
  if (disjoint && sine_splits(a.N, tiles(16))) {
    if (a.N <= 1024 && tiles(16) * ((pairs + 3) / 4) < SINE_CHAIN_WGS) {
      if (sine_chain_ok(a, ROWS)) return sine_chain_launch<T, ROWS>(a, fs, tiles(16), pairs, st);
      return sine_launch<T, ROWS, 1, 1, 4>(a, fs, tiles(16), pairs, 4, st);
    }
    return sine_launch<T, ROWS, 1, 1>(a, fs, tiles(16), (pairs + 3) / 4, 4, st);
  }
  if (pairs > 64) return ST_UNSUPPORTED;  // in place: one work-group holds every output of a tile
  const bool wide = tiles(32) >= 512;
  if (pairs <= 16)
    return wide ? sine_launch<T, ROWS, 1, 2>(a, fs, tiles(32), 1, pairs, st)
                : sine_launch<T, ROWS, 1, 1>(a, fs, tiles(16), 1, pairs, st);
  if (pairs <= 32)
    return wide ? sine_launch<T, ROWS, 2, 2>(a, fs, tiles(32), 1, (pairs + 1) / 2, st)
                : sine_launch<T, ROWS, 2, 1>(a, fs, tiles(16), 1, (pairs + 1) / 2, st);
  return sine_launch<T, ROWS, 4, 1>(a, fs, tiles(16), 1, (pairs + 3) / 4, st);
}

template <typename T, bool ROWS, int KS> int sine_jobs_launch(SineJobs<T>& s, int blocks, int nmax, hipStream_t st) {
  s.mc = sine_mc(nmax, 16, KS > 1);
  const size_t lds = sine_lds_bytes<T, ROWS, 1>(nmax, s.mc);
  static std::once_flag once;
  TRY_ST(sine_lds(&k_dst_sine_jobs<T, ROWS, KS, 0>, lds, once));
  hipLaunchKernelGGL((k_dst_sine_jobs<T, ROWS, KS, 0>), dim3(blocks), dim3(256), lds, st, s);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}
template <typename T, bool ROWS> int sine_jobs_chain(SineJobs<T>& s, int blocks, int nmax, hipStream_t st) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), sine_chain_lds<T>(nmax), st, s);
  };
  if (nmax <= 128) launch(k_dst_sine_jobs<T, ROWS, 4, 4>);
  else launch(k_dst_sine_jobs<T, ROWS, 4, 8>);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

// Strided pencils so short that 16 x 16 products are mostly padding (N < 32 fills one pair of
// them): one thread per output has no more to do, and transforms, scales and transforms back in one
// launch and one trip to memory where the products take two.  The pass along the slowest axis of a
// solve, products against one thread per output, FP64: 300 x 200 columns of 4, 9, 13, 17 and 20
// intervals, of the whole solve 64 and 47, 88 and 74, 102 and 89, 117 and 108, 126 and 123 us; 150 x
// 50 of 7 and 13 40.5 and 38.5, 40.9 and 41.5.  Two plain passes along y: 300 x 200 columns of 4, 9
// and 13 intervals 62 and 52, 86 and 79, 97 and 98; 160 x 50 of 7 40.0 and 40.8.  In FP32 the lines lie
// at the same bytes a row of columns.
template <typename T> bool short_pencils(int N, long long columns, bool fused) {
  const bool wide = columns * (long long)sizeof(T) >= 200000;
  return fused ? N < (wide ? 18 : 12) : N < (wide ? 12 : 6);
}

}  // namespace

template <typename T>
int dst_direct_pass(int N, const T* sn2, const T* in, T* out, long long outer, long long inner, long long pitch,
                    const DstScale<T>* fused, hipStream_t st, T* tmp, int cols) {
  if (N < 2 || N > DST_MAX_N || !sn2 || !in || !out || outer < 0 || inner < 1) return ST_INVALID;
  const int L = N - 1;
  if (inner == 1 && (pitch < L || fused)) return ST_INVALID;
  if (cols < L) cols = L;
  // (the output pairs reach the next multiple of 32)
  if (inner == 1 && cols > L && (cols > pitch || cols > (N / 2 + 15) / 16 * 32)) return ST_INVALID;
  if (outer == 0) return ST_OK;
  if (inner == 1 || !short_pencils<T>(N, outer * inner, fused != nullptr)) {
    const long long extent = inner == 1 ? (outer - 1) * pitch + cols : outer * (long long)L * inner;
    auto apart = [&](const T* x, const T* y) { return x + extent <= y || y + extent <= x; };
    auto run = [&](const T* src, T* dst, const DstScale<T>* f) {
      SineArgs<T> s;
      s.in = src;
      s.out = dst;
      s.sn = sn2;
      s.N = N;
      s.half = 0;
      s.cols = cols;
      s.outer = outer;
      s.inner = inner;
      s.pitch = pitch;
      return inner == 1 ? sine_pass<T, true>(s, f, apart(src, dst), st)
                        : sine_pass<T, false>(s, f, apart(src, dst), st);
    };
    T* mid = tmp && apart(in, tmp) && apart(out, tmp) ? tmp : out;
    int rc = run(in, fused ? mid : out, fused);
    if (rc == ST_OK && fused) rc = run(mid, out, nullptr);
    if (rc != ST_UNSUPPORTED) return rc;  // refused before anything is launched
  }
  const size_t per = (size_t)L * sizeof(T) * 2;  // x and y of one pencil
  int P = (int)std::min<size_t>(64, std::max<size_t>(1, (48 * 1024) / per));
  if ((size_t)P * per > DIRECT_LDS_MAX) return ST_UNSUPPORTED;
  DirectArgs<T> a;
  a.in = in;
  a.out = out;
  a.sn2 = sn2;
  a.N = N;
  a.P = P;
  a.outer = outer;
  a.inner = inner;
  a.pitch = pitch;
  a.cols = cols;
  a.fused = fused != nullptr;
  if (fused) a.fs = *fused;
  long long blocks;
  if (inner == 1) {
    a.ntile_inner = 1;
    blocks = (outer + P - 1) / P;
  } else {
    a.ntile_inner = (inner + P - 1) / P;
    blocks = outer * a.ntile_inner;
  }
  if (blocks > 0x7fffffffLL) return ST_UNSUPPORTED;
  const size_t lds = (size_t)P * per;
  if (lds > 64 * 1024) set_direct_lds_attr<T>();
  hipLaunchKernelGGL(k_dst_direct<T>, dim3((unsigned)blocks), dim3(256), lds, st, a);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

bool dst_direct_splits(int N, long long outer, long long inner) {
  return sine_splits(N, inner == 1 ? (outer + 15) / 16 : outer * ((inner + 15) / 16));
}

// Flops of a pass as sine products, its pencils rounded up to the tile.
double dst_sine_flops(int N, long long outer, long long inner) {
  const double pencils = inner == 1 ? (double)((outer + 15) / 16 * 16) : (double)outer * ((inner + 15) / 16 * 16);
  return pencils * N * N;
}

template <typename T> int dst_sine_jobs(const SineJob<T>* jobs, int count, hipStream_t st) {
  if (count < 1) return ST_OK;
  const bool rows = jobs[0].inner == 1;
  for (int j0 = 0; j0 < count; j0 += SINE_JOBS_MAX) {
    SineJobs<T> s;
    int nmax = 0;
    const int n = std::min(SINE_JOBS_MAX, count - j0);
    long long tiles[SINE_JOBS_MAX] = {0}, wg = 0;
    for (int j = 0; j < SINE_JOBS_MAX; ++j) {
      const SineJob<T>& q = jobs[j0 + std::min(j, n - 1)];
      SineArgs<T>& a = s.job[j];
      a.in = q.in;
      a.out = q.out;
      a.sn = q.tb->sn;
      a.N = q.tb->N;
      a.half = q.tb->ppt != 0;
      a.cols = a.N - 1;
      if (a.N > DST_SINE_JOBS_MAX_N) return ST_UNSUPPORTED;
      a.outer = q.outer;
      a.inner = q.inner;
      a.pitch = q.pitch;
      if (!a.sn || (q.inner == 1) != rows || (rows && q.pitch < a.N - 1)) return ST_INVALID;
      a.ntile_inner = rows ? 1 : (q.inner + 15) / 16;
      s.groups[j] = (a.N / 2 + 15) / 16;  // pairs
      if (j < n) tiles[j] = rows ? (q.outer + 15) / 16 : q.outer * a.ntile_inner;
      wg += tiles[j] * ((s.groups[j] + 3) / 4);
      nmax = std::max(nmax, a.N);
    }
    const bool chain = wg < SINE_CHAIN_WGS;
    bool direct = chain;
    for (int j = 0; j < n; ++j) direct = direct && sine_chain_ok(s.job[j], rows);
    long long blocks = 0;
    for (int j = 0; j < SINE_JOBS_MAX; ++j) {
      if (!chain) s.groups[j] = (s.groups[j] + 3) / 4;
      blocks += tiles[j] * s.groups[j];
      if (blocks > 0x7fffffffLL) return ST_UNSUPPORTED;
      s.end[j] = (int)blocks;
    }
    if (blocks == 0) continue;
    if (direct) TRY_ST((rows ? sine_jobs_chain<T, true>(s, (int)blocks, nmax, st) : sine_jobs_chain<T, false>(s, (int)blocks, nmax, st)));
    else if (rows) TRY_ST(chain ? sine_jobs_launch<T, true, 4>(s, (int)blocks, nmax, st) : sine_jobs_launch<T, true, 1>(s, (int)blocks, nmax, st));
    else TRY_ST(chain ? sine_jobs_launch<T, false, 4>(s, (int)blocks, nmax, st) : sine_jobs_launch<T, false, 1>(s, (int)blocks, nmax, st));
  }
  return ST_OK;
}
template int dst_sine_jobs<float>(const SineJob<float>*, int, hipStream_t);
template int dst_sine_jobs<double>(const SineJob<double>*, int, hipStream_t);

template int dst_direct_pass<float>(int, const float*, const float*, float*, long long, long long, long long,
                                    const DstScale<float>*, hipStream_t, float*, int);
template int dst_direct_pass<double>(int, const double*, const double*, double*, long long, long long, long long,
                                     const DstScale<double>*, hipStream_t, double*, int);

}  // namespace ahoc
