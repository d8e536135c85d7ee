// DST-I along both axes of every plane of a 3-D array in one launch (gfx950), both axes of
// DST_PLANE_MAX_N intervals or fewer.
//
// Two passes over a small grid cost two launches, two trips to memory and two ramps up and down
// of the chip, each several times the time its bytes take (128^3 in FP64: 13 and 15 us for
// 33 MB of cache traffic, 6 us).  Here a work-group takes 16 R values of y's transform of one
// plane over its whole length in x, keeps them in LDS and transforms them along x.  A plane is
// split over the work-groups by the parity of y's index first: with
// sin(pi k (N-m) / N) = (-1)^(k+1) sin(pi k m / N) odd and even outputs are half-size sums over
// y_m + y_{N-m} and y_m - y_{N-m}, so each work-group runs half the products on folded
// inputs, and 127 planes give 508 work-groups where whole planes would fill half the chip.  The
// transform is its own inverse up to a factor and the axes commute: the same kernel runs both
// directions.  It reads elsewhere than it writes (the work-groups of a plane all read it), the
// caller's dense FP64 rows too, which takes the copies to and from padded rows out.
//
// Both sums run on the matrix cores in the working precision (sine operand gathered from the
// period tables in LDS).  A wavefront's 16 columns of the first sum are its own, so their
// operand comes straight from memory to registers, folded there; the tile is folded over x
// before the second sum reads it.  The work-groups of a plane sit on one XCD: the plane's second
// to fourth read hit its L2.
//
// A Dirichlet solve between dense arrays, a pass per axis against planes (and the slowest axis in
// one launch to 96), FP64 and FP32: 128^3 98 -> 61 and 71 -> 50 us, 99 x 89 x 74 points 65 -> 52 and
// 53 -> 39, 96^3 69 -> 49 and 57 -> 37, 64^3 32 -> 21 and 32 -> 19, 48^3 51 -> 20 and 48 -> 18, 32^3
// 29 -> 18 and 29 -> 17.  FP32 errors against 64 bits (rms of a solve): 128^3 5.8e-7 -> 5.1e-7, 64^3
// 3.7e-7 -> 3.0e-7, 99 x 89 x 74 points 4.0e-7 -> 3.6e-7.  A pass at 128^3 in FP64 takes 20 us: 7 of
// matrix-core time, 5 of the other vector instructions, 3 of LDS and the trips to memory, in phases
// that the two work-groups of a CU run side by side.
#include "common.h"
#include "mfma_sine.h"

#include <algorithm>

namespace ahoc {

namespace {

template <typename T> struct PlaneArgs {
  const T* sn[2];  // sin(pi j / n), j = 0..2n-1, or (half, even n) j = 0..n/2; axis 0: x, 1: y
  int half[2];
  int n[2];
  long long in_pitch, out_pitch;
  int out_cols;  // columns written per row: n[0] - 1, or more (zeros) up to the pitch
  int planes;
  int parts;     // work-groups of a plane: 2 * groups of 16 R outputs of one parity
};

// Values of the tile row in LDS (32 pairs of outputs, conflict-free like the sine passes' rows)
template <typename T> __host__ __device__ constexpr int plane_ld(int pairs) { return 32 * pairs + SineOps<T>::PAD; }

// First period-table indices and their steps of four values of m for outputs k (odd) and k + 1
// (even) of lane group lk; outputs beyond N - 1 take index 0.
__device__ __forceinline__ unsigned sine_wrap(unsigned i, unsigned two_n) { return min(i, i - two_n); }  // i < 2 two_n
__device__ __forceinline__ void sine_indices(unsigned k, int N, int lk, unsigned* ie, unsigned* io, unsigned* de,
                                             unsigned* dd) {
  const unsigned two_n = 2u * N, ke = (int)k < N ? k : 0u, ko = (int)k + 1 < N ? k + 1u : 0u;
  *ie = sine_wrap(ke * (1u + lk), two_n);
  *io = sine_wrap(ko * (1u + lk), two_n);
  *de = sine_wrap(4u * ke, two_n);
  *dd = sine_wrap(4u * ko, two_n);
}

// K: steps of four values of m that cover y's half length.
template <typename T, typename TI, typename TO, int R, int K>
__global__ void __launch_bounds__(512) k_dst_plane(PlaneArgs<T> a, const TI* __restrict__ in, TO* __restrict__ out) {
  using S = SineOps<T>;
  using v4 = typename S::v4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int plane = ((int)blockIdx.x >> 3) / a.parts * 8 + ((int)blockIdx.x & 7);
  if (plane >= a.planes) return;
  const int part = ((int)blockIdx.x >> 3) % a.parts;
  const int par = part & 1, g0 = (part >> 1) * 16 * R;  // outputs 2 (g0 + i) + 1 + par of y
  const int N0 = a.n[0], N1 = a.n[1], L0 = N0 - 1, L1 = N1 - 1, H0 = N0 / 2, H1 = N1 / 2;
  const int nt = blockDim.x, pairs = nt >> 7, ld = plane_ld<T>(pairs);
  T* tile = reinterpret_cast<T*>(smem);
  T* t0 = tile + 16 * R * ld;
  T* t1 = t0 + sine_pad(2 * N0);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const TI* src = in + (long long)plane * L1 * a.in_pitch;

  // this wavefront's columns, folded over y: values m = 4 s + lk + 1 of column x
  const int x = 16 * w + li;
  T f[K];
  {
    // all K steps are within H1 but the last two (all four of K = 4): those load a clamped row
    // and count as zero beyond H1.  Columns x >= L0 carry the last column's values to nowhere.
    constexpr int SAFE = K > 4 ? K - 2 : 0;
    const unsigned pitch = (unsigned)a.in_pitch * sizeof(TI), xc = min(x, L0 - 1) * sizeof(TI);  // bytes
    auto at = [&](unsigned off) { return *reinterpret_cast<const TI*>(reinterpret_cast<const char*>(src) + off); };
    TI u[K], v[K];
    const T s0 = sine_entry<T>(a.sn[0], N0, a.half[0], min((int)threadIdx.x, 2 * N0 - 1));
    const T s1 = sine_entry<T>(a.sn[1], N1, a.half[1], min((int)threadIdx.x, 2 * N1 - 1));
    const unsigned up = lk * pitch + xc, down = (L1 - 1 - lk) * pitch + xc;  // rows m - 1 and N1 - m - 1
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int m = 4 * s + lk + 1;
      u[s] = at(s < SAFE || m <= H1 ? up + 4u * s * pitch : xc);
      v[s] = at(s < SAFE || m <= H1 ? down - 4u * s * pitch : xc);
    }
    if ((int)threadIdx.x < 2 * N0) t0[sine_pad(threadIdx.x)] = s0;
    if ((int)threadIdx.x < 2 * N1) t1[sine_pad(threadIdx.x)] = s1;
    for (int i = threadIdx.x + nt; i < 2 * N0; i += nt) t0[sine_pad(i)] = sine_entry<T>(a.sn[0], N0, a.half[0], i);
    for (int i = threadIdx.x + nt; i < 2 * N1; i += nt) t1[sine_pad(i)] = sine_entry<T>(a.sn[1], N1, a.half[1], i);
    const T sign = par ? T(-1) : T(1);
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int m = 4 * s + lk + 1;
      const T vs = s < SAFE || 2 * m != N1 ? T(v[s]) : T(0);
      const T e = T(u[s]) + sign * vs;
      f[s] = s < SAFE || m <= H1 ? e : T(0);
    }
  }
  __syncthreads();
  {
    const unsigned two_n = 2u * N1;
    unsigned idx[R], step[R];
    v4 acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      unsigned k = 2u * (g0 + 16 * r + li) + 1u + par;
      k = (int)k < N1 ? k : 0u;  // no such output
      idx[r] = sine_wrap(k * (1u + lk), two_n);
      step[r] = sine_wrap(4u * k, two_n);
      acc[r] = v4{T(0), T(0), T(0), T(0)};
    }
#pragma unroll
    for (int s = 0; s < K; ++s)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        acc[r] = S::mfma(t1[sine_pad(idx[r])], f[s], acc[r]);
        idx[r] = sine_wrap(idx[r] + step[r], two_n);
      }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) tile[(16 * r + S::row(lk, q)) * ld + x] = acc[r][q];
  }
  __syncthreads();
  // fold over x in place: e_m = t_m + t_{N-m} in the first half of a row, o_m = t_m - t_{N-m} in
  // the second, zeros beyond H0 (four values of m per thread: 16 R rows of 16 pairs)
  const int half = 16 * pairs;
  {
    constexpr int FW = 2 * R;
    const int row0 = ((int)threadIdx.x >> 4) / pairs, m = (int)threadIdx.x - row0 * half + 1, mc = min(m, H0);
    T* t = tile + row0 * ld;
    T e[FW], o[FW];
#pragma unroll
    for (int j = 0; j < FW; ++j) {
      const T u = t[8 * j * ld + mc - 1], v = t[8 * j * ld + N0 - mc - 1];
      const T vs = 2 * m == N0 ? T(0) : v;
      e[j] = m > H0 ? T(0) : u + vs;
      o[j] = m > H0 ? T(0) : u - vs;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < FW; ++j) {
      t[8 * j * ld + m - 1] = e[j];
      t[8 * j * ld + half + m - 1] = o[j];
    }
  }
  __syncthreads();
  // along x: outputs 32 p + 2 li (+ 1) of rows r16 = (w & 1), (w & 1) + 2, ..
  const int p = w >> 1;
  constexpr int RW = R / 2;
  const unsigned two_n = 2u * N0;
  unsigned ie, io, de, dd;
  sine_indices(32u * p + 2u * li + 1u, N0, lk, &ie, &io, &de, &dd);
  v4 ae[RW], ao[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) ae[r] = ao[r] = v4{T(0), T(0), T(0), T(0)};
  const T* row = tile + (16 * (w & 1) + li) * ld + lk;
  for (int s0 = 0; s0 < H0; s0 += 16, row += 16) {  // the tile is zero up to the next multiple of 16
#pragma unroll
    for (int s = 0; s < 16; s += 4) {
      const T se = t0[sine_pad(ie)], so = t0[sine_pad(io)];
      ie = sine_wrap(ie + de, two_n);
      io = sine_wrap(io + dd, two_n);
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        ae[r] = S::mfma(row[32 * r * ld + s], se, ae[r]);
        ao[r] = S::mfma(row[32 * r * ld + half + s], so, ao[r]);
      }
    }
  }
  const int k = 32 * p + 2 * li;
  TO* dst = out + (long long)plane * L1 * a.out_pitch;
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int y = 2 * (g0 + 16 * ((w & 1) + 2 * r) + S::row(lk, q)) + par;
      if (y >= L1) continue;
      TO* o = dst + (unsigned)(y * (int)a.out_pitch + k);
      if (k < a.out_cols) o[0] = k < L0 ? TO(ae[r][q]) : TO(0);
      if (k + 1 < a.out_cols) o[1] = k + 1 < L0 ? TO(ao[r][q]) : TO(0);
    }
}

// The slowest axis of a solve in place: transform, eigen scaling, transform back, 16 columns per
// work-group of one wavefront per pair of 16 odd and 16 even outputs.  The columns stay in LDS in
// between, where the separate sine passes cross memory (99 x 89 x 74 points in FP64: two launches
// of 9 us); the generic FFT kernel, one thread row per pencil pair with a radix loop, took 28 us
// at 47^3.
template <typename T>
__global__ void __launch_bounds__(256)
    k_dst_solve_sine(T* data, const T* __restrict__ sn, int half_table, int N, long long inner, DstScale<T> fs) {
  using S = SineOps<T>;
  using v4 = typename S::v4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nt = blockDim.x, half = nt >> 2, L = N - 1, H = N / 2;
  T* x = reinterpret_cast<T*>(smem);  // [2 half][16]
  T* tab = x + 2 * half * 16;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const long long c0 = blockIdx.x * 16LL, col = c0 + li;
  const bool in = col < inner;
  constexpr int FW = 4;  // values of m per thread: 16 * half / nt
  T e[FW], o[FW], st[8];
  {
    T u[FW], v[FW];
    const T* src = data + (in ? col : inner - 1);
    const T s0 = sine_entry<T>(sn, N, half_table, min((int)threadIdx.x, 2 * N - 1));
#pragma unroll
    for (int j = 0; j < FW; ++j) {
      const int m = min((threadIdx.x >> 4) + j * (nt >> 4) + 1, (unsigned)H);
      u[j] = src[(m - 1) * inner];
      v[j] = src[(N - m - 1) * inner];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // eigenvalues of this lane's outputs
      const int k = 32 * w + 2 * S::row(lk, q);
      st[2 * q] = fs.s_this[min(k, L - 1)];
      st[2 * q + 1] = fs.s_this[min(k + 1, L - 1)];
    }
    if ((int)threadIdx.x < 2 * N) tab[sine_pad(threadIdx.x)] = s0;
    for (int i = threadIdx.x + nt; i < 2 * N; i += nt) tab[sine_pad(i)] = sine_entry<T>(sn, N, half_table, i);
#pragma unroll
    for (int j = 0; j < FW; ++j) {
      const int m = (threadIdx.x >> 4) + j * (nt >> 4) + 1;
      const T vs = 2 * m == N ? T(0) : v[j];
      e[j] = in && m <= H ? u[j] + vs : T(0);
      o[j] = in && m <= H ? u[j] - vs : T(0);
    }
  }
  T A = 1, B = 0;
  {
    const long long ib = col / fs.na;
    const long long ia = col - ib * fs.na;
    if (in && ia < fs.nva) {
      const T sa = fs.s_a[ia];
      const T sb = fs.s_b ? fs.s_b[ib] : T(0);
      A = sa + sb + fs.c_ab * sa * sb + fs.a0 + fs.ka * sa + fs.kb * sb;
      B = T(1) + fs.c_ta * sa + fs.c_tb * sb + fs.kt;
    }
  }
  const unsigned two_n = 2u * N;
  unsigned ie0, io0, de, dd;
  sine_indices(32u * w + 2u * li + 1u, N, lk, &ie0, &io0, &de, &dd);
#pragma unroll 1
  for (int turn = 0; turn < 2; ++turn) {
#pragma unroll
    for (int j = 0; j < FW; ++j) {  // [m][16]: e below, o above
      x[threadIdx.x + j * nt] = e[j];
      x[16 * half + threadIdx.x + j * nt] = o[j];
    }
    __syncthreads();
    v4 ae = v4{T(0), T(0), T(0), T(0)}, ao = ae;
    unsigned ie = ie0, io = io0;
    const T* xe = x + lane;
    const T* xo = xe + 16 * half;
    for (int s0 = 0; s0 < H; s0 += 16, xe += 256, xo += 256) {  // zeros up to the next multiple of 16
#pragma unroll
      for (int s = 0; s < 16; s += 4) {
        const T se = tab[sine_pad(ie)], so = tab[sine_pad(io)];
        ie = sine_wrap(ie + de, two_n);
        io = sine_wrap(io + dd, two_n);
        ae = S::mfma(se, xe[16 * s], ae);
        ao = S::mfma(so, xo[16 * s], ao);
      }
    }
    if (turn) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 32 * w + 2 * S::row(lk, q);
        T* out = data + k * inner + col;
        if (in && k < L) out[0] = ae[q];
        if (in && k + 1 < L) out[inner] = ao[q];
      }
      return;
    }
    __syncthreads();  // the products' reads are done
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 32 * w + 2 * S::row(lk, q);
      x[16 * k + li] = ae[q] * (fs.scale / (A + B * st[2 * q]));
      x[16 * k + 16 + li] = ao[q] * (fs.scale / (A + B * st[2 * q + 1]));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < FW; ++j) {
      const int m = (threadIdx.x >> 4) + j * (nt >> 4) + 1, mc = min(m, H);
      const T u = x[16 * (mc - 1) + li], v = x[16 * (N - mc - 1) + li];
      const T vs = 2 * m == N ? T(0) : v;
      e[j] = m <= H ? u + vs : T(0);
      o[j] = m <= H ? u - vs : T(0);
    }
    __syncthreads();
  }
}

}  // namespace

template <typename T>
int dst_solve_axis(const DstTables<T>& tb, T* data, long long inner, long long pitch, const DstScale<T>& fs, int tile,
                   T* tmp, hipStream_t st) {
  // The length-specialised FFT kernel is ahead from 128 on, its pass longer below: a solve, FFT
  // against products here, 128^3 63.3 and 66.0 us in FP64, 50.7 and 52.9 in FP32; 96^3 53.3 and
  // 50.4, 44.0 and 37.0; 64^3 22.2 and 21.4, 21.5 and 18.4; 32^3 18.0 and 16.6, 18.6 and 16.6.
  if (tb.N > DST_PLANE_MAX_N || (tb.N > 96 && dst_fast_supported(tb.N)))
    return dst_pass<T>(tb, data, data, 1, inner, pitch, &fs, tile, st, nullptr, tmp);
  if (tb.N < 4 || !tb.sn || !data || inner < 1) return ST_INVALID;
  const long long blocks = (inner + 15) / 16;
  if (blocks > 0x7fffffffLL) return ST_UNSUPPORTED;
  const int pairs = (tb.N / 2 + 15) / 16;
  const size_t lds = sizeof(T) * (512 * (size_t)pairs + sine_pad(2 * tb.N));
  hipLaunchKernelGGL(k_dst_solve_sine<T>, dim3((unsigned)blocks), dim3(64 * pairs), lds, st, data, tb.sn, tb.ppt != 0,
                     tb.N, inner, fs);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}
template int dst_solve_axis<float>(const DstTables<float>&, float*, long long, long long, const DstScale<float>&, int,
                                   float*, hipStream_t);
template int dst_solve_axis<double>(const DstTables<double>&, double*, long long, long long, const DstScale<double>&,
                                    int, double*, hipStream_t);

bool dst_plane_ok(int n0, int n1) { return n0 >= 4 && n1 >= 4 && n0 <= DST_PLANE_MAX_N && n1 <= DST_PLANE_MAX_N; }

// A plane takes the time of 32 outputs of either parity of y for each 32 columns of x, whatever its
// size in y, where the time of separate passes goes with its values once they outlast their
// launches.  A solve, separate passes against planes, FP64: 128 x 8 points in y of 256, 512, 2048
// planes 42 and 40, 51 and 63, 124 and 189 us; 128 x 16 of 512 and 2048 planes 59 and 56, 157 and
// 203; 128 x 32 of 2048 planes 266 and 242; 64 x 8 and 64 x 16 of 2048 planes 88 and 100, 110 and
// 105; 32 x 8 of 2048 planes 71 and 65; 8 x 8 of 4096 planes 96 and 101.  The two meet at y = 8 per
// 32 columns of x in long grids (twice that where x fills less than half of them), below it where
// fewer than some thousand groups of columns leave the launches as the time.
bool dst_plane_pays(int n0, int n1, int planes) {
  const long long pairs = (n0 / 2 + 15) / 16;
  return dst_plane_ok(n0, n1) && n1 >= std::min((n0 < 16 ? 16 : 8) * pairs, planes * pairs / 128);
}

template <typename T, typename TI, typename TO>
int dst_plane_pass(const DstTables<T>& tx, const DstTables<T>& ty, const TI* in, long long in_pitch, TO* out,
                   long long out_pitch, int planes, hipStream_t st) {
  const int L0 = tx.N - 1, L1 = ty.N - 1;
  if (!dst_plane_ok(tx.N, ty.N) || !tx.sn || !ty.sn || !in || !out || in_pitch < L0 || out_pitch < L0 || planes < 0 ||
      L1 * std::max(in_pitch, out_pitch) > 0x1fffffffLL)
    return ST_INVALID;
  if (planes == 0) return ST_OK;
  constexpr int R = 2;  // R = 4 (half the work-groups): 32 to 128 planes slower, 128 x 128 x 31 points 47 us for 35
  const int pairs = (tx.N / 2 + 15) / 16;
  PlaneArgs<T> a;
  a.sn[0] = tx.sn;
  a.sn[1] = ty.sn;
  a.half[0] = tx.ppt != 0;
  a.half[1] = ty.ppt != 0;
  a.n[0] = tx.N;
  a.n[1] = ty.N;
  a.in_pitch = in_pitch;
  a.out_pitch = out_pitch;
  a.out_cols = (int)std::min<long long>(out_pitch, 32 * pairs);
  a.planes = planes;
  a.parts = 2 * ((ty.N / 2 + 16 * R - 1) / (16 * R));
  const long long blocks = (planes + 7LL) / 8 * 8 * a.parts;
  if (blocks > 0x7fffffffLL) return ST_UNSUPPORTED;
  const size_t lds = sizeof(T) * (16 * R * (size_t)plane_ld<T>(pairs) + sine_pad(2 * tx.N) + sine_pad(2 * ty.N));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(128 * pairs), lds, st, a, in, out);
  };
  const int k = (ty.N / 2 + 3) / 4;
  if (k <= 4) launch(k_dst_plane<T, TI, TO, R, 4>);
  else if (k <= 6) launch(k_dst_plane<T, TI, TO, R, 6>);
  else if (k <= 8) launch(k_dst_plane<T, TI, TO, R, 8>);
  else if (k <= 10) launch(k_dst_plane<T, TI, TO, R, 10>);
  else if (k <= 12) launch(k_dst_plane<T, TI, TO, R, 12>);
  else if (k <= 14) launch(k_dst_plane<T, TI, TO, R, 14>);
  else launch(k_dst_plane<T, TI, TO, R, 16>);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}
#define AHOC_PLANE(T, TI, TO)                                                                                       \
  template int dst_plane_pass<T, TI, TO>(const DstTables<T>&, const DstTables<T>&, const TI*, long long, TO*,       \
                                         long long, int, hipStream_t);
AHOC_PLANE(double, double, double)
AHOC_PLANE(float, float, float)
AHOC_PLANE(float, double, float)
AHOC_PLANE(float, float, double)
#undef AHOC_PLANE

}  // namespace ahoc
