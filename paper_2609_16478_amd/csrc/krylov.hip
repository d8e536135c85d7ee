// FP64 Krylov kernels of the device-resident GMRES(m) (matrix-free GMRES on
// S_h Q = b, Sec. 2.3).  Arnoldi uses classical Gram-Schmidt with one
// re-orthogonalisation (two block dot-product sweeps instead of j dependent
// ones), Givens rotations keep the least-squares residual |g_{j+1}|.
// Reductions are two-stage with a fixed order, so results are reproducible.
#include "common.h"
#include "kernels.h"

#include <algorithm>

namespace ahoc {

namespace {

constexpr int TPB = 256;

__device__ __forceinline__ double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// Every kernel works on `ns` independent segments (the instances of a batch, 1 for a
// single problem): a vector of the Krylov basis is ns consecutive segments of length n,
// and each segment has its own dot products, Hessenberg matrix, rotations and norms.
// Per-segment small arrays: H [ns][m][m+1] (column j at j*(m+1)), cs, sn [ns][m],
// gv, y, h1, h2 [ns][m+1], nrm, resid [ns][2], beta [ns], act [ns].

// part[(s * nvec + v) * gridDim.x + block] = partial sum of <V_v, w> over segment s, or with
// one block per segment and `out` given, the sum itself at out[s * ostride + v].  The
// vectors are taken MDC at a time, so that w is read once per group of vectors rather than
// once per vector; each vector's sum runs over the same elements in the same order either way.
constexpr int MDC = 8;
// Sums of eight per-lane values over a wavefront: halves of the lanes exchange halves of the
// values, so that 4 + 2 + 1 + 3 shuffles do what eight butterflies would take 48 for (the
// shuffles of FP64 pairs, not the sums, are what a short sweep waits for).  The lane whose bits
// 5, 4, 3 spell c ends up with the sum of value c.
static_assert(MDC == 8, "wave_sum8 reduces groups of eight");
__device__ __forceinline__ double wave_sum8(double (&a)[MDC], int lane) {
#pragma unroll
  for (int half = 4, bit = 32; half >= 1; half >>= 1, bit >>= 1) {
    const bool up = lane & bit;
#pragma unroll
    for (int c = 0; c < half; ++c) {
      const double send = up ? a[c] : a[c + half];
      const double keep = up ? a[c + half] : a[c];
      a[c] = keep + __shfl_xor(send, bit, 64);
    }
  }
  a[0] += __shfl_xor(a[0], 4, 64);
  a[0] += __shfl_xor(a[0], 2, 64);
  a[0] += __shfl_xor(a[0], 1, 64);
  return a[0];
}
// The group's MDC sums are reduced together: across each wavefront with shuffles, then the
// TPB/64 wavefront sums added in wavefront order by one thread per vector (one barrier per
// group; the LDS rows alternate between groups, so a group's rows are not overwritten before
// they are read).
__global__ void k_mdot_partial(const double* __restrict__ V, long long ld, int nvec,
                               const double* __restrict__ w, long long n, double* __restrict__ part,
                               double* __restrict__ out, int ostride) {
  constexpr int NW = TPB / 64;
  __shared__ double red[2][NW][MDC];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const long long s0 = blockIdx.y * n;
  const double* ws = w + s0;
  for (int v0 = 0; v0 < nvec; v0 += MDC) {
    const int nv = nvec - v0 < MDC ? nvec - v0 : MDC;
    double acc[MDC];
#pragma unroll
    for (int c = 0; c < MDC; ++c) acc[c] = 0;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
         e += (long long)gridDim.x * blockDim.x) {
      const double we = ws[e];
#pragma unroll
      for (int c = 0; c < MDC; ++c)
        if (c < nv) acc[c] += V[(long long)(v0 + c) * ld + s0 + e] * we;
    }
    const double sum = wave_sum8(acc, lane);
    const int buf = (v0 / MDC) & 1;
    if ((lane & 7) == 0) red[buf][wv][lane >> 3] = sum;
    __syncthreads();
    if (threadIdx.x < nv) {
      const int c = threadIdx.x;
      double r = red[buf][0][c];
#pragma unroll
      for (int k = 1; k < NW; ++k) r += red[buf][k][c];
      if (out) out[(long long)blockIdx.y * ostride + v0 + c] = r;
      else part[((long long)blockIdx.y * nvec + v0 + c) * gridDim.x + blockIdx.x] = r;
    }
  }
}

// out[s * ostride + v] (+)= sum of the partials of (segment s, vector v)
__global__ void k_mdot_reduce(const double* __restrict__ part, int nbk, int nvec, double* __restrict__ out,
                              int ostride, int accumulate) {
  __shared__ double red[TPB];
  const int v = blockIdx.x;
  const long long sg = blockIdx.y;
  double acc = 0;
  for (int b = threadIdx.x; b < nbk; b += blockDim.x) acc += part[(sg * nvec + v) * nbk + b];
  const double r = block_sum(acc, red);
  if (threadIdx.x == 0) {
    double* o = out + sg * ostride + v;
    *o = accumulate ? *o + r : r;
  }
}

// w_s += sign * sum_v coef[s * cstride + v] V_v  on each segment s
__global__ void k_maxpy(double* __restrict__ w, const double* __restrict__ V, long long ld, int nvec,
                        const double* __restrict__ coef, int cstride, double sign, long long n) {
  const long long s0 = blockIdx.y * n;
  const double* c = coef + (long long)blockIdx.y * cstride;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    double acc = 0;
    for (int v = 0; v < nvec; ++v) acc += c[v] * V[(long long)v * ld + s0 + e];
    w[s0 + e] += sign * acc;
  }
}

__global__ void k_axpby(long long n, double a, const double* __restrict__ x, double b, double* __restrict__ y) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    y[e] = b == 0.0 ? a * x[e] : a * x[e] + b * y[e];
}

// The sums of a and b over a work-group of TPB threads, in every thread, in a fixed order.
__device__ __forceinline__ void block_sum2(double& a, double& b, double (*red)[TPB / 64]) {
  for (int m = 32; m >= 1; m >>= 1) {
    a += __shfl_xor(a, m, 64);
    b += __shfl_xor(b, m, 64);
  }
  __syncthreads();  // red is free
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = a;
    red[1][threadIdx.x >> 6] = b;
  }
  __syncthreads();
  a = red[0][0];
  b = red[1][0];
#pragma unroll
  for (int q = 1; q < TPB / 64; ++q) {
    a += red[0][q];
    b += red[1][q];
  }
}

// BiCGSTAB's vector steps (kernels.h).  Every work-group adds the parts of the dot products up
// itself: a few thousand values from L2 instead of a reduction launch, a copy to the host and a
// wait for it.  What bounds them is memory: at 128^3 (16.5 MB a vector, in the last-level cache)
// the half step takes 10 us, 4.7 TB/s, the full one 23 us, 5.7 TB/s.  A solve with variable beta
// at 128^3, 35 iterations in all, 14.0 -> 10.3 ms with them, the dot products in the operator's
// kernel and two waits an iteration instead of four.
__global__ void __launch_bounds__(TPB)
    k_bicg_half(long long n, double rho, const double* __restrict__ part, int nb1, const double* __restrict__ v,
                double* __restrict__ r, double* __restrict__ coef, double* __restrict__ part2) {
  __shared__ double red[2][TPB / 64];
  double d = 0, rr = 0;
  for (int b = threadIdx.x; b < nb1; b += TPB) d += part[b];
  block_sum2(d, rr, red);
  const bool good = d != 0.0 && isfinite(d);
  const double alpha = good ? rho / d : 0.0;
  rr = 0;
  if (good)
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
         e += (long long)gridDim.x * blockDim.x) {
      const double x = r[e] - alpha * v[e];
      r[e] = x;
      rr += x * x;
    }
  double zero = 0;
  block_sum2(rr, zero, red);
  if (threadIdx.x == 0) {
    part2[blockIdx.x] = rr;
    if (blockIdx.x == 0) {
      coef[0] = alpha;
      coef[1] = good ? 1.0 : 0.0;
    }
  }
}

__global__ void __launch_bounds__(TPB)
    k_bicg_full(long long n, const double* __restrict__ part, int nb1, const double* __restrict__ y,
                const double* __restrict__ z, const double* __restrict__ t, const double* __restrict__ rh,
                double* __restrict__ x, double* __restrict__ r, double* __restrict__ coef,
                double* __restrict__ part2) {
  __shared__ double red[2][TPB / 64];
  double st = 0, tt = 0;
  for (int b = threadIdx.x; b < nb1; b += TPB) {
    st += part[b];
    tt += part[nb1 + b];
  }
  block_sum2(st, tt, red);
  const bool good = tt != 0.0 && isfinite(st / tt);
  const double alpha = coef[0], omega = good ? st / tt : 0.0;
  double hr = 0, rr = 0;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x) {
    if (good) {
      x[e] = alpha * y[e] + omega * z[e] + x[e];
      const double v = r[e] - omega * t[e];
      r[e] = v;
      hr += rh[e] * v;
      rr += v * v;
    } else {
      x[e] = alpha * y[e] + x[e];
    }
  }
  block_sum2(hr, rr, red);
  if (threadIdx.x == 0) {
    part2[blockIdx.x] = hr;
    part2[gridDim.x + blockIdx.x] = rr;
    if (blockIdx.x == 0) {
      coef[2] = omega;
      coef[3] = good ? 1.0 : 0.0;
    }
  }
}

__global__ void __launch_bounds__(TPB)
    k_bicg_to_host(const double* __restrict__ part, int nb, int nvec, const double* __restrict__ coef,
                   double* __restrict__ out) {
  __shared__ double red[2][TPB / 64];
  double a = 0, b = 0;
  for (int q = threadIdx.x; q < nb; q += TPB) {
    a += part[q];
    if (nvec > 1) b += part[nb + q];
  }
  block_sum2(a, b, red);
  if (threadIdx.x == 0) {
    out[0] = a;
    if (nvec > 1) out[1] = b;
  }
  if (threadIdx.x < 4) out[4 + threadIdx.x] = coef[threadIdx.x];
}

// w = a x + b y + c w
__global__ void k_lin3(long long n, double a, const double* __restrict__ x, double b, const double* __restrict__ y,
                       double c, double* __restrict__ w) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    w[e] = a * x[e] + b * y[e] + c * w[e];
}

// x_s = 0 on every segment s with keep[s] == 0
__global__ void k_zero_masked(double* __restrict__ x, long long n, const int* __restrict__ keep) {
  if (keep[blockIdx.y]) return;
  const long long s0 = blockIdx.y * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    x[s0 + e] = 0.0;
}

// out_s = src[s] (or 0 where src[s] is null): concatenate per-instance arrays of length n
__global__ void k_gather_ptrs(const double* const* __restrict__ src, long long n, double* __restrict__ out) {
  const double* p = src[blockIdx.y];
  double* o = out + blockIdx.y * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    o[e] = p ? p[e] : 0.0;
}

// dst[s] = in_s: split a batch array into per-instance arrays of length n
__global__ void k_scatter_ptrs(const double* __restrict__ in, long long n, double* const* __restrict__ dst) {
  double* p = dst[blockIdx.y];
  const double* x = in + blockIdx.y * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    p[e] = x[e];
}

// one wavefront per segment: y_s[0..k_s) from the rotated triangle by columns (a solved y_i
// leaves the right-hand sides above it, spread over the lanes), y_s[k_s..kmax) = 0
__global__ void k_back_solve(const double* H, int m, const double* gv, const int* kk, int kmax, double* y) {
  constexpr int PER = 4;  // entries per lane: m <= 256
  const int sg = blockIdx.x, lane = threadIdx.x;
  const int ldh = m + 1;
  const double* Hs = H + (long long)sg * m * ldh;
  const double* g_ = gv + (long long)sg * ldh;
  double* ys = y + (long long)sg * ldh;
  const int k = kk[sg];
  double t[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = lane + 64 * q;
    t[q] = i < k ? g_[i] : 0.0;
    if (i < kmax) ys[i] = 0.0;
  }
  for (int i = k - 1; i >= 0; --i) {
    const double* col = Hs + (long long)i * ldh;
    double h[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) h[q] = lane + 64 * q <= i ? col[lane + 64 * q] : 0.0;
    double yi = 0.0;
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (q == i / 64) yi = __shfl(t[q] / h[q], i & 63, 64);
#pragma unroll
    for (int q = 0; q < PER; ++q)
      if (lane + 64 * q < i) t[q] -= h[q] * yi;
    if (lane == (i & 63)) ys[i] = yi;
  }
}

__global__ void k_start(double* __restrict__ v0, const double* __restrict__ r, long long n,
                        const double* __restrict__ nrm2, double* gv, int m, double* beta) {
  const long long sg = blockIdx.y;
  const double b = sqrt(fmax(nrm2[2 * sg], 0.0));
  const double ib = b > 0 ? 1.0 / b : 0.0;
  const long long s0 = sg * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    v0[s0 + e] = r[s0 + e] * ib;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double* g_ = gv + sg * (m + 1);
    g_[0] = b;
    for (int i = 1; i <= m; ++i) g_[i] = 0.0;
    beta[sg] = b;
  }
}

// The rest of Arnoldi step j of one segment, by one work-group: the column h[0..j] = <V_i, w>
// (both sweeps) and the norm nn of the new vector, rotated by the earlier rotations, give the
// next rotation and the residual estimate |g_{j+1}|; then the per-instance bookkeeping, on the
// device, so that the host need not read the estimates every step.  ist = [act | kk | nit |
// flag | hcnt] (ns ints each): the (active) instance counts the step, records its Krylov
// dimension j + 1 and stops -- flag 1 -- when |g_{j+1}| <= tol ||b||, with flag 2 when the
// estimate is not finite or, for an FP32 operator (inexact), when eight steps gained less
// than a factor 2 below 1e-2 (ring of its last 16 estimates in hist), and without a flag at
// the iteration cap.  eres keeps each instance's estimate of its last active step.
struct ArnoldiState {
  double *H, *cs, *sn, *gv, *resid;
  const double* bnorm;
  int* ist;
  double *hist, *eres;
  double tol;
  int ns, m, j, max_iters, inexact;
};
constexpr int ARN_MAX_M = 200;  // longest restart length (ahoc_setup clamps to it)
// The state the end of the step reads, fetched before its norm is known (each of these loads
// would otherwise be one more memory round trip of a single thread).
struct ArnoldiLds {
  double c[ARN_MAX_M], s[ARN_MAX_M];
  double g, bnorm, old;
  int nit, hcnt, still;
};
__device__ __forceinline__ void prefetch_state(const ArnoldiState& a, int sg, ArnoldiLds& l) {
  for (int i = threadIdx.x; i < a.j; i += blockDim.x) {
    l.c[i] = a.cs[(long long)sg * a.m + i];
    l.s[i] = a.sn[(long long)sg * a.m + i];
  }
  if (threadIdx.x == 64) l.g = a.gv[(long long)sg * (a.m + 1) + a.j];
  if (threadIdx.x == 65) l.bnorm = a.bnorm[sg];
  if (threadIdx.x == 66) l.nit = a.ist[2 * a.ns + sg];
  if (threadIdx.x == 67) {
    l.hcnt = a.ist[4 * a.ns + sg];
    l.old = a.hist[16LL * sg + ((l.hcnt + 1 - 9) & 15)];
  }
}
// h: LDS, overwritten; every thread of the work-group calls it, after a barrier since
// prefetch_state and the writes of h.  Returns whether the segment stays active.
__device__ __forceinline__ bool rotate_and_update(const ArnoldiState& a, int sg, double* h, ArnoldiLds& l, double nn) {
  const int j = a.j, ldh = a.m + 1;
  if (threadIdx.x == 0) {
    double lo = h[0];
    for (int i = 0; i < j; ++i) {
      const double hi = h[i + 1], c = l.c[i], s = l.s[i];
      h[i] = c * lo + s * hi;
      lo = -s * lo + c * hi;
    }
    const double rho = hypot(lo, nn);
    const double c = rho > 0 ? lo / rho : 1.0, s = rho > 0 ? nn / rho : 0.0;
    h[j] = rho;
    double* g_ = a.gv + (long long)sg * ldh;
    const double gj = l.g, res = fabs(-s * gj), est = res / l.bnorm;
    const int it = l.nit + 1;
    int flag = 0;
    bool stop = false;
    if (!isfinite(est)) {
      flag = 2;
      stop = true;
    } else if (est <= a.tol) {
      flag = 1;
      stop = true;
    } else {
      if (a.inexact) {
        const int hc = l.hcnt + 1;
        a.hist[16LL * sg + ((hc - 1) & 15)] = est;
        a.ist[4 * a.ns + sg] = hc;
        if (hc > 8 && est < 1e-2 && est > 0.5 * l.old) {
          flag = 2;
          stop = true;
        }
      }
      if (it >= a.max_iters) stop = true;
    }
    a.cs[(long long)sg * a.m + j] = c;
    a.sn[(long long)sg * a.m + j] = s;
    g_[j + 1] = -s * gj;
    g_[j] = c * gj;
    a.resid[2 * sg] = res;
    a.resid[2 * sg + 1] = nn;
    a.eres[sg] = est;
    a.ist[a.ns + sg] = j + 1;
    a.ist[2 * a.ns + sg] = it;
    if (flag) a.ist[3 * a.ns + sg] = flag;
    if (stop) a.ist[sg] = 0;
    l.still = !stop;
  }
  __syncthreads();
  double* col = a.H + (long long)sg * a.m * ldh + (long long)j * ldh;
  for (int i = threadIdx.x; i <= j + 1; i += blockDim.x) col[i] = i <= j ? h[i] : 0.0;
  return l.still;
}

// One Arnoldi step of a short segment (n <= NT EPT) in one work-group: w = V_{j+1} holds the
// operator's output; both Gram-Schmidt sweeps, the norm, the rotation with the bookkeeping and
// the scaling.  w and the first NV basis vectors stay in registers, fetched in one round trip;
// later vectors are read from the caches four times.  Latency bound throughout: a sweep is two
// barriers, one after all its wavefront sums and one after their totals.  At 1596 unknowns (13
// vectors on average) 19 us; the seven launches of the step written as separate sweeps 52 us.
// A segment that is no longer active gets w = 0.
template <int NT, int EPT, int NV>
__global__ void __launch_bounds__(NT) k_arnoldi_one(double* __restrict__ V, long long ld, long long n,
                                                    ArnoldiState a) {
  constexpr int NW = NT / 64;
  static_assert(NV % MDC == 0, "the register basis is summed in groups of eight");
  __shared__ double red[ARN_MAX_M + MDC][NW];
  __shared__ double h1[ARN_MAX_M + 1], hs[ARN_MAX_M + 1];
  __shared__ ArnoldiLds l;
  const int sg = blockIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nvec = a.j + 1;
  const long long s0 = sg * n;
  double* wp = V + (long long)nvec * ld + s0;
  const bool act = a.ist[sg] != 0;
  // entries past n read the last one; their w stays 0
  int at[EPT];
  double w[EPT], vr[NV][EPT];
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    at[q] = min(threadIdx.x + NT * q, (int)n - 1);
    w[q] = threadIdx.x + NT * q < n ? wp[at[q]] : 0.0;
  }
#pragma unroll
  for (int v0 = 0; v0 < NV; v0 += MDC) {
    if (v0 < nvec) {
#pragma unroll
      for (int c = 0; c < MDC; ++c) {
        const double* vp = V + (long long)min(v0 + c, nvec - 1) * ld + s0;
#pragma unroll
        for (int q = 0; q < EPT; ++q) vr[v0 + c][q] = vp[at[q]];
      }
    }
  }
  if (!act) {
#pragma unroll
    for (int q = 0; q < EPT; ++q)
      if (threadIdx.x + NT * q < n) wp[at[q]] = 0.0;
    return;
  }
  prefetch_state(a, sg, l);
#pragma unroll 1
  for (int sweep = 0; sweep < 2; ++sweep) {
    double* h = sweep ? hs : h1;
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += MDC) {
      if (v0 < nvec) {
        double acc[MDC];
#pragma unroll
        for (int c = 0; c < MDC; ++c) {
          acc[c] = 0;
#pragma unroll
          for (int q = 0; q < EPT; ++q) acc[c] += vr[v0 + c][q] * w[q];
        }
        const double sum = wave_sum8(acc, lane);
        if ((lane & 7) == 0) red[v0 + (lane >> 3)][wv] = sum;
      }
    }
    for (int v0 = NV; v0 < nvec; v0 += MDC) {
      double acc[MDC];
#pragma unroll
      for (int c = 0; c < MDC; ++c) {
        acc[c] = 0;
        const double* vp = V + (long long)min(v0 + c, nvec - 1) * ld + s0;
#pragma unroll
        for (int q = 0; q < EPT; ++q) acc[c] += vp[at[q]] * w[q];
      }
      const double sum = wave_sum8(acc, lane);
      if ((lane & 7) == 0) red[v0 + (lane >> 3)][wv] = sum;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < nvec; v += NT) {
      double r = red[v][0];
#pragma unroll
      for (int k = 1; k < NW; ++k) r += red[v][k];
      h[v] = r;
    }
    __syncthreads();
    double d[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) d[q] = 0;
#pragma unroll
    for (int v0 = 0; v0 < NV; v0 += MDC) {
      if (v0 < nvec) {
#pragma unroll
        for (int c = 0; c < MDC; ++c) {
          const double hv = v0 + c < nvec ? h[v0 + c] : 0.0;
#pragma unroll
          for (int q = 0; q < EPT; ++q) d[q] += hv * vr[v0 + c][q];
        }
      }
    }
#pragma unroll 4
    for (int v = NV; v < nvec; ++v) {
      const double* vp = V + (long long)v * ld + s0;
      const double hv = h[v];
#pragma unroll
      for (int q = 0; q < EPT; ++q) d[q] += hv * vp[at[q]];
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q) w[q] = threadIdx.x + NT * q < n ? w[q] - d[q] : 0.0;
  }
  double nn = 0;
#pragma unroll
  for (int q = 0; q < EPT; ++q) nn += w[q] * w[q];
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) nn += __shfl_xor(nn, m, 64);
  // red and h1 are free: their last reads, the totals of the second sweep and the update of the
  // first, lie before a barrier that every wavefront has passed.  hs is not: a slower wavefront
  // may still be in its second update, so the column is summed in h1.
  if (lane == 0) red[0][wv] = nn;
  for (int i = threadIdx.x; i < nvec; i += NT) h1[i] += hs[i];
  __syncthreads();
  nn = red[0][0];
#pragma unroll
  for (int k = 1; k < NW; ++k) nn += red[0][k];
  nn = sqrt(fmax(nn, 0.0));
  const bool still = rotate_and_update(a, sg, h1, l, nn);
  const double r = nn > 0 && still ? 1.0 / nn : 0.0;
#pragma unroll
  for (int q = 0; q < EPT; ++q)
    if (threadIdx.x + NT * q < n) wp[at[q]] = w[q] * r;
}

// The same step of a longer segment, over gridDim.x slices of it (gridDim.y segments).  Every
// work-group sums the partial dot products of the launch before by itself where they are few
// (hin null; the sums in slice order, the same in every work-group), so that a step is four
// launches instead of eleven: 35 instead of 55 us at 97 thousand unknowns.
//
// w -= sum_v h_v V_v over the slice, h the sums of part (or hin), kept in hout by slice 0; then
// the partial dot products <V_v, w> of the new w (sweep 1) or its partial <w, w> (sweep 2) into
// part2.  A slice is at most ARN_SLICE entries, held in LDS between the two.
constexpr int ARN_SLICE = 2048;  // the most that arnoldi_slices gives
__device__ __forceinline__ void sum_partials(const double* __restrict__ part, int nbk, int nvec, int sg,
                                             double* __restrict__ h) {
  constexpr int U = 4;  // vectors in flight per wavefront
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int v0 = wv; v0 < nvec; v0 += U * nw) {
    double r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      r[u] = 0;
      const int v = min(v0 + u * nw, nvec - 1);
      for (int b = lane; b < nbk; b += 64) r[u] += part[((long long)sg * nvec + v) * nbk + b];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) r[u] += __shfl_xor(r[u], m, 64);
      if (lane == 0 && v0 + u * nw < nvec) h[v0 + u * nw] = r[u];
    }
  }
}
template <bool SECOND>
__global__ void __launch_bounds__(TPB) k_arnoldi_update(double* __restrict__ V, long long ld, long long n, int nvec,
                                                        const double* __restrict__ part,
                                                        const double* __restrict__ hin, double* __restrict__ hout,
                                                        int m, double* __restrict__ part2,
                                                        const int* __restrict__ act, int* __restrict__ act0) {
  constexpr int NW = TPB / 64;
  __shared__ double h[ARN_MAX_M + 1];
  __shared__ double red[2][NW][MDC];
  __shared__ double ws[ARN_SLICE];
  const int sg = blockIdx.y, nbk = gridDim.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // the flag as the step found it, for the last launch, whose slice 0 changes it
  if (SECOND && blockIdx.x == 0 && threadIdx.x == 0) act0[sg] = act[sg];
  if (!act[sg]) return;  // the last launch writes w = 0
  const long long per = (n + nbk - 1) / nbk, lo = blockIdx.x * per, s0 = sg * n + lo;
  const int cnt = (int)(n - lo < per ? (n - lo > 0 ? n - lo : 0) : per);
  if (hin) {
    for (int v = threadIdx.x; v < nvec; v += TPB) h[v] = hin[(long long)sg * (m + 1) + v];
  } else {
    sum_partials(part, nbk, nvec, sg, h);
  }
  __syncthreads();
  if (blockIdx.x == 0 && !hin)
    for (int v = threadIdx.x; v < nvec; v += TPB) hout[(long long)sg * (m + 1) + v] = h[v];
  double* wp = V + (long long)nvec * ld + s0;
  double norm = 0;
  for (int e = threadIdx.x; e < cnt; e += TPB) {
    double d = 0;
#pragma unroll 8
    for (int v = 0; v < nvec; ++v) d += h[v] * V[(long long)v * ld + s0 + e];
    const double x = wp[e] - d;
    wp[e] = x;
    if (SECOND) norm += x * x;
    else ws[e] = x;  // read back by this thread only
  }
  for (int v0 = 0; v0 < (SECOND ? 1 : nvec); v0 += MDC) {
    const int nv = SECOND ? 1 : (nvec - v0 < MDC ? nvec - v0 : MDC);
    double acc[MDC];
#pragma unroll
    for (int c = 0; c < MDC; ++c) acc[c] = 0;
    if (SECOND) {
      acc[0] = norm;
    } else {
      for (int e = threadIdx.x; e < cnt; e += TPB) {
        const double x = ws[e];
#pragma unroll
        for (int c = 0; c < MDC; ++c)
          if (c < nv) acc[c] += V[(long long)(v0 + c) * ld + s0 + e] * x;
      }
    }
    const double sum = wave_sum8(acc, lane);
    const int buf = (v0 / MDC) & 1;
    if ((lane & 7) == 0) red[buf][wv][lane >> 3] = sum;
    __syncthreads();
    if (threadIdx.x < nv) {
      double r = red[buf][0][threadIdx.x];
#pragma unroll
      for (int k = 1; k < NW; ++k) r += red[buf][k][threadIdx.x];
      part2[((long long)sg * (SECOND ? 1 : nvec) + v0 + threadIdx.x) * nbk + blockIdx.x] = r;
    }
  }
}

// The end of the step: the norm from the nbk partials of the second sweep (or nrm2[2 sg]), w scaled by it
// slice by slice, the rotation and the bookkeeping by slice 0.  The vector of the step at which
// a segment stops is scaled like the others (it is in no column that the solution reads); from
// the next step on the segment's vectors are zero.
__global__ void __launch_bounds__(TPB) k_arnoldi_finish(double* __restrict__ V, long long ld, long long n, int nbk,
                                                        const double* __restrict__ part,
                                                        const double* __restrict__ nrm2,
                                                        const double* __restrict__ h1, const double* __restrict__ h2,
                                                        const int* __restrict__ act0, ArnoldiState a) {
  __shared__ double hs[ARN_MAX_M + 1], nsum[1];
  __shared__ ArnoldiLds l;
  const int sg = blockIdx.y, nvec = a.j + 1;
  double* wp = V + (long long)nvec * ld + sg * n;
  const bool act = act0[sg] != 0;
  double r = 0.0;
  if (act) {
    if (blockIdx.x == 0) {
      prefetch_state(a, sg, l);
      for (int i = threadIdx.x; i < nvec; i += TPB)
        hs[i] = h1[(long long)sg * (a.m + 1) + i] + h2[(long long)sg * (a.m + 1) + i];
    }
    if (!nrm2) sum_partials(part, nbk, 1, sg, nsum);
    __syncthreads();
    const double nn = sqrt(fmax(nrm2 ? nrm2[2 * sg] : nsum[0], 0.0));
    r = nn > 0 ? 1.0 / nn : 0.0;
    if (blockIdx.x == 0) rotate_and_update(a, sg, hs, l, nn);
  }
  for (long long e = blockIdx.x * (long long)TPB + threadIdx.x; e < n; e += (long long)gridDim.x * TPB)
    wp[e] = act ? wp[e] * r : 0.0;
}

__global__ void k_fill_int(int* __restrict__ p, long long n, int v) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    p[e] = v;
}

inline unsigned nblk(long long n, int cap) {
  long long b = (n + TPB - 1) / TPB;
  if (b > cap) b = cap;
  return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

int mdot_partial(const double* V, long long ld, int nvec, const double* w, long long n, int ns, double* part,
                 int nbk, hipStream_t st) {
  hipLaunchKernelGGL(k_mdot_partial, dim3(nbk, ns), dim3(TPB), 0, st, V, ld, nvec, w, n, part, nullptr, 0);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int mdot(const double* V, long long ld, int nvec, const double* w, long long n, int ns, double* part, int nbk,
         double* out, int ostride, hipStream_t st) {
  if (nbk == 1) {  // one block per segment: its sum is the result (no reduction launch)
    hipLaunchKernelGGL(k_mdot_partial, dim3(1, ns), dim3(TPB), 0, st, V, ld, nvec, w, n, part, out, ostride);
    AHOC_HIP_TRY(hipGetLastError());
    return ST_OK;
  }
  TRY_ST(mdot_partial(V, ld, nvec, w, n, ns, part, nbk, st));
  return mdot_reduce(part, nbk, nvec, ns, out, ostride, 0, st);
}

int mdot_reduce(const double* part, int nbk, int nvec, int ns, double* out, int ostride, int accumulate,
                hipStream_t st) {
  hipLaunchKernelGGL(k_mdot_reduce, dim3(nvec, ns), dim3(TPB), 0, st, part, nbk, nvec, out, ostride, accumulate);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int maxpy(double* w, const double* V, long long ld, int nvec, const double* coef, int cstride, double sign,
          long long n, int ns, hipStream_t st) {
  hipLaunchKernelGGL(k_maxpy, dim3(nblk(n, 65536), ns), dim3(TPB), 0, st, w, V, ld, nvec, coef, cstride, sign, n);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int axpby(long long n, double a, const double* x, double b, double* y, hipStream_t st) {
  hipLaunchKernelGGL(k_axpby, dim3(nblk(n, 65536)), dim3(TPB), 0, st, n, a, x, b, y);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int bicg_half(long long n, double rho, const double* part, int nb1, const double* v, double* r, double* coef,
              double* part2, int nb2, hipStream_t st) {
  hipLaunchKernelGGL(k_bicg_half, dim3(nb2), dim3(TPB), 0, st, n, rho, part, nb1, v, r, coef, part2);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int bicg_full(long long n, const double* part, int nb1, const double* y, const double* z, const double* t,
              const double* rh, double* x, double* r, double* coef, double* part2, int nb2, hipStream_t st) {
  hipLaunchKernelGGL(k_bicg_full, dim3(nb2), dim3(TPB), 0, st, n, part, nb1, y, z, t, rh, x, r, coef, part2);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int bicg_to_host(const double* part, int nb, int nvec, const double* coef, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_bicg_to_host, dim3(1), dim3(TPB), 0, st, part, nb, nvec, coef, out);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int lin3(long long n, double a, const double* x, double b, const double* y, double c, double* w, hipStream_t st) {
  hipLaunchKernelGGL(k_lin3, dim3(nblk(n, 65536)), dim3(TPB), 0, st, n, a, x, b, y, c, w);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int zero_masked(double* x, long long n, int ns, const int* keep, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_masked, dim3(nblk(n, 65536), ns), dim3(TPB), 0, st, x, n, keep);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int gather_ptrs(const double* const* src, long long n, int ns, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_ptrs, dim3(nblk(n, 65536), ns), dim3(TPB), 0, st, src, n, out);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int scatter_ptrs(const double* in, long long n, int ns, double* const* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_scatter_ptrs, dim3(nblk(n, 65536), ns), dim3(TPB), 0, st, in, n, dst);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int back_solve(int ns, const double* H, int m, const double* gv, const int* kk, int kmax, double* y,
               hipStream_t st) {
  if (m > 256) return ST_UNSUPPORTED;
  hipLaunchKernelGGL(k_back_solve, dim3(ns), dim3(64), 0, st, H, m, gv, kk, kmax, y);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

// Slices of a long segment: 512 entries each (two per thread: the sweeps are latency-bound)
// while every work-group can still sum their partials itself, else 2048.
int arnoldi_slices(long long n) {
  const long long b = (n + 511) / 512;
  return (int)(b <= ARN_INLINE ? b : std::max<long long>(ARN_INLINE, (n + ARN_SLICE - 1) / ARN_SLICE));
}

int arnoldi_step(double* V, long long ld, long long n, const ArnoldiArgs& g, hipStream_t st) {
  if (g.m > ARN_MAX_M || g.j >= g.m) return ST_INVALID;
  const int nvec = g.j + 1;
  ArnoldiState a{g.H, g.cs, g.sn, g.gv, g.resid, g.bnorm, g.ist, g.hist, g.eres, g.tol, g.ns, g.m, g.j, g.max_iters,
                 g.inexact ? 1 : 0};
  if (n <= ARN_ONE_MAX) {
    static_assert(ARN_ONE_MAX <= 512 * 4, "the last kernel's entries");
    const dim3 grid(g.ns);
    if (n <= 512) hipLaunchKernelGGL((k_arnoldi_one<512, 1, 32>), grid, dim3(512), 0, st, V, ld, n, a);
    else if (n <= 1024) hipLaunchKernelGGL((k_arnoldi_one<512, 2, 32>), grid, dim3(512), 0, st, V, ld, n, a);
    else hipLaunchKernelGGL((k_arnoldi_one<512, 4, 16>), grid, dim3(512), 0, st, V, ld, n, a);
    AHOC_HIP_TRY(hipGetLastError());
    return ST_OK;
  }
  const int nbk = arnoldi_slices(n);
  if ((n + nbk - 1) / nbk > ARN_SLICE) return ST_UNSUPPORTED;
  const bool few = nbk <= ARN_INLINE;
  const dim3 grid(nbk, g.ns);
  double* p1 = g.part;
  double* p2 = p1 + (long long)g.ns * (g.m + 1) * nbk;
  double* w = V + (long long)nvec * ld;
  hipLaunchKernelGGL(k_mdot_partial, grid, dim3(TPB), 0, st, V, ld, nvec, w, n, p1, nullptr, 0);
  if (!few) TRY_ST(mdot_reduce(p1, nbk, nvec, g.ns, g.h1, g.m + 1, 0, st));
  hipLaunchKernelGGL((k_arnoldi_update<false>), grid, dim3(TPB), 0, st, V, ld, n, nvec, p1, few ? nullptr : g.h1,
                     g.h1, g.m, p2, g.ist, g.act0);
  if (!few) TRY_ST(mdot_reduce(p2, nbk, nvec, g.ns, g.h2, g.m + 1, 0, st));
  hipLaunchKernelGGL((k_arnoldi_update<true>), grid, dim3(TPB), 0, st, V, ld, n, nvec, p2, few ? nullptr : g.h2,
                     g.h2, g.m, p1, g.ist, g.act0);
  if (!few) TRY_ST(mdot_reduce(p1, nbk, 1, g.ns, g.nrm, 2, 0, st));
  hipLaunchKernelGGL(k_arnoldi_finish, dim3((unsigned)std::min<long long>(2048, (n + 1023) / 1024), g.ns), dim3(TPB),
                     0, st, V, ld, n, nbk, p1, few ? nullptr : g.nrm, g.h1, g.h2, g.act0, a);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int fill_int(int* p, long long n, int v, hipStream_t st) {
  if (n <= 0) return ST_OK;
  hipLaunchKernelGGL(k_fill_int, dim3(nblk(n, 4096)), dim3(TPB), 0, st, p, n, v);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int start_cycle(double* v0, const double* r, long long n, int ns, const double* nrm2, double* gv, int m,
                double* beta, hipStream_t st) {
  hipLaunchKernelGGL(k_start, dim3(nblk(n, 65536), ns), dim3(TPB), 0, st, v0, r, n, nrm2, gv, m, beta);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

}  // namespace ahoc
