// Grid-stencil kernels of the augmented scheme (gfx950).
//
//   lift      G = src + L_h^bnd[Q]      right-hand side of the v-equation
//                                       (-L_h V = M f, V = Q on face interiors)
//   rhs_u     G = src + M(V / alpha)    right-hand side of the u-equation, with
//                                       V = Q on the face-interior nodes M reaches
//   gather    R = alpha_b h^-2 (6 U1 - 3/2 U2 + 2/9 U3) - Q - src_q
//                                       boundary residual of Lemma 1 (one-sided
//                                       normal formula of Sec. 2.2, known data in src_q)
//   resid64   FP64 residual of the coupled system (iterative refinement)
//   setup     1/alpha, alpha on faces, M f and the data lifts
//
// All are memory-bound streaming kernels: one thread per node, neighbours come
// through L1/L2.  Interior arrays use the working precision T; data, the
// refinement state and the Krylov vectors are FP64.
#include "common.h"
#include "kernels.h"

namespace ahoc {

namespace {

constexpr int TPB = 256;

// launch sizes of the row-based traversals: one work-group per interior / nodal row
inline unsigned interior_rows(const Geom& g) {
  return (unsigned)(g.dim == 3 ? (long long)g.ni[1] * g.ni[2] : g.ni[1]);
}
inline unsigned nodal_rows(const Geom& g) {
  return (unsigned)(g.dim == 3 ? (long long)g.nn[1] * g.nn[2] : g.nn[1]);
}

inline unsigned nblocks(long long n) {
  long long b = (n + TPB - 1) / TPB;
  if (b > 1048576) b = 1048576;
  return (unsigned)(b < 1 ? 1 : b);
}

__device__ __forceinline__ long long nod(const Geom& g, int i, int j, int k) {
  return ((long long)k * g.nn[1] + j) * g.nn[0] + i;
}
__device__ __forceinline__ long long inr(const Geom& g, int i, int j, int k) {
  return ((long long)(k - 1) * g.ni[1] + (j - 1)) * g.px + (i - 1);
}

// number of coordinates of node (i,j,k) on the boundary
template <int DIM> __device__ __forceinline__ int nbnd(const Geom& g, int i, int j, int k) {
  int c = (i == 0 || i == g.n[0]) + (j == 0 || j == g.n[1]);
  if (DIM == 3) c += (k == 0 || k == g.n[2]);
  return c;
}

// Q index of a face-interior node.
template <int DIM> __device__ __forceinline__ int qidx(const Geom& g, int i, int j, int k) {
  if (i == 0 || i == g.n[0]) {
    const int f = (i == 0) ? 0 : 1;
    return g.face_off[f] + (DIM == 3 ? (k - 1) * g.ni[1] : 0) + (j - 1);
  }
  if (j == 0 || j == g.n[1]) {
    const int f = (j == 0) ? 2 : 3;
    return g.face_off[f] + (DIM == 3 ? (k - 1) * g.ni[0] : 0) + (i - 1);
  }
  const int f = (k == 0) ? 4 : 5;
  return g.face_off[f] + (j - 1) * g.ni[0] + (i - 1);
}

// decode Q index -> boundary node, face axis and inward step
template <int DIM>
__device__ __forceinline__ void dec_q(const Geom& g, int q, int& i, int& j, int& k, int& axis, int& step) {
  int f = 0;
  while (f + 1 < 2 * DIM && q >= g.face_off[f + 1]) ++f;
  const int t = q - g.face_off[f];
  axis = f >> 1;
  const int side = f & 1;
  step = side ? -1 : 1;
  const int fix = side ? g.n[axis] : 0;
  if (DIM == 2) {
    k = 0;
    if (axis == 0) { i = fix; j = t + 1; }
    else { j = fix; i = t + 1; }
  } else {
    if (axis == 0) { i = fix; j = t % g.ni[1] + 1; k = t / g.ni[1] + 1; }
    else if (axis == 1) { j = fix; i = t % g.ni[0] + 1; k = t / g.ni[0] + 1; }
    else { k = fix; i = t % g.ni[0] + 1; j = t / g.ni[0] + 1; }
  }
}

// weight of L_h at offset (dx, dy, dz); 0 for offsets outside the compact stencil
template <int DIM> __device__ __forceinline__ double lw(const Weights& w, int dx, int dy, int dz) {
  const int nz = (dx != 0) + (dy != 0) + (dz != 0);
  if (nz == 0) return w.c0;
  if (nz == 1) return dx ? w.cf[0] : (dy ? w.cf[1] : w.cf[2]);
  if (nz == 2) {
    if (DIM == 2) return w.ce[0];
    return dz == 0 ? w.ce[0] : (dy == 0 ? w.ce[1] : w.ce[2]);
  }
  return 0.0;
}

// ---------------------------------------------------------------------------------
template <typename T, int DIM>
__global__ void k_lift(Geom g, Weights w, const T* __restrict__ Q, const T* __restrict__ src,
                       T* __restrict__ G) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  Q += b_ * g.nq;
  if (src) src += b_ * g.nalloc;
  G += b_ * g.nalloc;
  // rows (j, k) across work-groups, x across threads (32-bit row decode)
  const int nrow_ = DIM == 3 ? g.ni[1] * g.ni[2] : g.ni[1];
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i0_ = threadIdx.x; i0_ < g.px; i0_ += blockDim.x) {
    const long long e = (long long)r_ * g.px + i0_;
    const int i = i0_ + 1, j = (DIM == 3 ? r_ % g.ni[1] : r_) + 1, k = DIM == 3 ? r_ / g.ni[1] + 1 : 0;
    if (i > g.ni[0]) {
      G[e] = T(0);
      continue;
    }
    T acc = src ? src[e] : T(0);
    const bool nearb = i == 1 || i == g.ni[0] || j == 1 || j == g.ni[1] ||
                       (DIM == 3 && (k == 1 || k == g.ni[2]));
    if (nearb) {
      const int zlo = DIM == 3 ? -1 : 0, zhi = DIM == 3 ? 1 : 0;
      for (int dz = zlo; dz <= zhi; ++dz)
        for (int dy = -1; dy <= 1; ++dy)
          for (int dx = -1; dx <= 1; ++dx) {
            const double wt = lw<DIM>(w, dx, dy, dz);
            if (wt == 0.0 || (dx == 0 && dy == 0 && dz == 0)) continue;
            const int qi = i + dx, qj = j + dy, qk = k + dz;
            if (nbnd<DIM>(g, qi, qj, qk) == 1) acc += (T)wt * Q[qidx<DIM>(g, qi, qj, qk)];
          }
    }
    G[e] = acc;
  }
}

// One work-group per interior row (j, k), threads along x: the row decode is two 32-bit
// integer operations per row instead of 64-bit divisions per node.
template <typename T, int DIM>
__global__ void k_rhs_u(Geom g, Weights w, const T* __restrict__ V, const T* __restrict__ Q,
                        const T* __restrict__ ia, const T* __restrict__ src, T* __restrict__ G) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  V += b_ * g.nalloc;
  Q += b_ * g.nq;
  ia += b_ * g.nnodal;
  if (src) src += b_ * g.nalloc;
  G += b_ * g.nalloc;
  const T m0 = (T)w.m0, m1 = (T)w.m1;
  const int nrow = DIM == 3 ? g.ni[1] * g.ni[2] : g.ni[1];
  for (int r = blockIdx.x; r < nrow; r += gridDim.x) {
    const int j = (DIM == 3 ? r % g.ni[1] : r) + 1;
    const int k = DIM == 3 ? r / g.ni[1] + 1 : 0;
    for (int i0 = threadIdx.x; i0 < g.px; i0 += blockDim.x) {
      const long long e = (long long)r * g.px + i0;
      const int i = i0 + 1;
      if (i > g.ni[0]) {
        G[e] = T(0);
        continue;
      }
      T acc = src ? src[e] : T(0);
      acc += m0 * V[e] * ia[nod(g, i, j, k)];
      T nb = 0;
#pragma unroll
      for (int a = 0; a < DIM; ++a)
#pragma unroll
        for (int s = -1; s <= 1; s += 2) {
          const int qi = i + (a == 0 ? s : 0), qj = j + (a == 1 ? s : 0), qk = k + (a == 2 ? s : 0);
          const bool bnd = (a == 0 && (qi == 0 || qi == g.n[0])) || (a == 1 && (qj == 0 || qj == g.n[1])) ||
                           (a == 2 && (qk == 0 || qk == g.n[2]));
          const T vq = bnd ? Q[qidx<DIM>(g, qi, qj, qk)] : V[inr(g, qi, qj, DIM == 3 ? qk : 1)];
          nb += vq * ia[nod(g, qi, qj, qk)];
        }
      G[e] = acc + m1 * nb;
    }
  }
}

// 3-D rhs_u: a work-group owns a tile of RBX x RBY columns and marches along z over kchunk
// planes.  W = V / alpha (on a face Q / alpha) of a thread's own column at planes k-1, k, k+1
// stays in registers, the next plane's value and its share of the tile's halo ring are
// prefetched, and the x- and y-neighbours come from an LDS copy of plane k (two copies in
// turn: one barrier per plane).  Memory bound: V, 1/alpha read (1 + 2/RBY + 2/kchunk) times.
// FP64: 14 us at 128^3 and 2.42 ms at 768^3 (4.5 TB/s of V, 1/alpha and G once each); whole
// rows of 512 threads over chunks of 32 planes took 121 us (128 work-groups with 3/4 of their
// threads idle) and 3.18 ms.
template <typename T>
__device__ __forceinline__ T w_at(const Geom& g, const T* __restrict__ V, const T* __restrict__ Q,
                                  const T* __restrict__ ia, int i, int j, int k) {
  // nodes with at most one boundary coordinate; 0 elsewhere (edges, past the far faces)
  const bool bi = i == 0 || i == g.n[0], bj = j == 0 || j == g.n[1], bk = k == 0 || k == g.n[2];
  if (i > g.n[0] || j > g.n[1] || k > g.n[2] || (int)bi + (int)bj + (int)bk > 1) return T(0);
  const T* p;
  if (bi) p = Q + g.face_off[i == 0 ? 0 : 1] + (long long)(k - 1) * g.ni[1] + (j - 1);
  else if (bj) p = Q + g.face_off[j == 0 ? 2 : 3] + (long long)(k - 1) * g.ni[0] + (i - 1);
  else if (bk) p = Q + g.face_off[k == 0 ? 4 : 5] + (long long)(j - 1) * g.ni[0] + (i - 1);
  else p = V + inr(g, i, j, k);
  return *p * ia[nod(g, i, j, k)];
}
constexpr int RBX = 64, RBY = 8;
template <typename T>
__global__ void __launch_bounds__(RBX * RBY) k_rhs_u_blk(Geom g, Weights w, const T* __restrict__ V,
                                                         const T* __restrict__ Q, const T* __restrict__ ia,
                                                         const T* __restrict__ src, T* __restrict__ G, int kchunk) {
  constexpr int RING = 2 * RBX + 2 * RBY;
  __shared__ T ws[2][RBY + 2][RBX + 2];
  const T m0 = (T)w.m0, m1 = (T)w.m1;
  const int ni1 = g.ni[1], ni2 = g.ni[2];
  const int tx = (g.px + RBX - 1) / RBX, ty = (ni1 + RBY - 1) / RBY, tz = (ni2 + kchunk - 1) / kchunk;
  const int total = tx * ty * tz;
  // work-groups are dealt round-robin to the 8 XCDs: give each XCD a contiguous range of
  // tiles, so that neighbouring tiles (sharing halo rows) meet in one L2
  const int per = (total + 7) / 8;
  const int idx = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
  if (blockIdx.x / 8 >= per || idx >= total) return;
  const int bx = idx % tx, by = idx / tx % ty, bz = idx / (tx * ty);
  const int lx = threadIdx.x % RBX, ly = threadIdx.x / RBX;
  const int i = bx * RBX + lx + 1, j = by * RBY + ly + 1;
  const int k0 = bz * kchunk + 1, k1 = min(ni2, k0 + kchunk - 1);
  // this thread's ring node (threads beyond the ring have none): the rows below and above the
  // tile, then the columns left and right of it
  const bool ring = threadIdx.x < RING;
  int hx = 0, hy = 0;
  if (threadIdx.x < 2 * RBX) {
    hx = lx + 1;
    hy = threadIdx.x < RBX ? 0 : RBY + 1;
  } else {
    const int r = threadIdx.x - 2 * RBX;
    hx = r < RBY ? 0 : RBX + 1;
    hy = r % RBY + 1;
  }
  const int hi = bx * RBX + hx, hj = by * RBY + hy;
  T wm = w_at(g, V, Q, ia, i, j, k0 - 1), wc = w_at(g, V, Q, ia, i, j, k0), wp = w_at(g, V, Q, ia, i, j, k0 + 1);
  T hv = ring ? w_at(g, V, Q, ia, hi, hj, k0) : T(0);
  for (int k = k0; k <= k1; ++k) {
    T(*row)[RBX + 2] = ws[k & 1];
    row[ly + 1][lx + 1] = wc;
    if (ring) row[hy][hx] = hv;
    __syncthreads();
    T wn = T(0);
    if (k < k1) {
      wn = w_at(g, V, Q, ia, i, j, k + 2);
      if (ring) hv = w_at(g, V, Q, ia, hi, hj, k + 1);
    }
    if (j <= ni1 && i <= g.px) {
      const long long e = ((long long)(k - 1) * ni1 + (j - 1)) * g.px + (i - 1);
      T acc = T(0);  // padding columns
      if (i <= g.ni[0]) {
        acc = m0 * wc + m1 * (row[ly + 1][lx] + row[ly + 1][lx + 2] + row[ly][lx + 1] + row[ly + 2][lx + 1] + wm + wp);
        if (src) acc += src[e];
      }
      G[e] = acc;
    }
    wm = wc;
    wc = wp;
    wp = wn;
  }
}

template <typename T, int DIM>
__global__ void k_gather(Geom g, Weights w, const T* __restrict__ U, const T* __restrict__ Q,
                         const T* __restrict__ af, const T* __restrict__ srcq, double* __restrict__ R) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  U += b_ * g.nalloc;
  Q += b_ * g.nq;
  af += b_ * g.nq;
  if (srcq) srcq += b_ * g.nq;
  R += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    T u[3];
#pragma unroll
    for (int m = 1; m <= 3; ++m) {
      const int ui = i + (ax == 0 ? st * m : 0), uj = j + (ax == 1 ? st * m : 0),
                uk = k + (ax == 2 ? st * m : 0);
      u[m - 1] = U[inr(g, ui, uj, DIM == 3 ? uk : 1)];
    }
    const T ih2 = (T)(1.0 / (g.h[ax] * g.h[ax]));
    T r = af[q] * ih2 * ((T)w.os[1] * u[0] + (T)w.os[2] * u[1] + (T)w.os[3] * u[2]) - Q[q];
    if (srcq) r -= srcq[q];
    R[q] = (double)r;
  }
}

// Face layers of the homogeneous lift L_h^bnd[Q]: the value at the interior node next to
// a face, taken from that face's own Q (its nodes inside the 19-point (3-D) or 9-point
// (2-D) stencil of the node), in the layouts of the spectral lift
//   3-D  Lx[s][(j-1) n_z' + (k-1)], Ly[s][(k-1) px + (i-1)], Lz[s][(j-1) px + (i-1)]
//   2-D  Lx[s][j-1], Ly[s][i-1]   (s = 0 low face, 1 high face; row padding zeroed)
// Each interior node's lift is the sum over the faces it touches.
template <int DIM>
__device__ __forceinline__ void face_node(const Geom& g, int f, long long t, int& i, int& j, int& k, int& valid) {
  const int ax = f >> 1, sd = f & 1;
  valid = 1;
  if (DIM == 2) {
    k = 0;
    if (ax == 0) {
      i = sd ? g.ni[0] : 1;
      j = (int)t + 1;
    } else {
      j = sd ? g.ni[1] : 1;
      i = (int)t + 1;
      valid = i <= g.ni[0];
    }
    return;
  }
  if (ax == 0) {  // [j][k]
    i = sd ? g.ni[0] : 1;
    j = (int)(t / g.ni[2]) + 1;
    k = (int)(t % g.ni[2]) + 1;
  } else if (ax == 1) {  // [k][i], pitch px
    j = sd ? g.ni[1] : 1;
    k = (int)(t / g.px) + 1;
    i = (int)(t % g.px) + 1;
    valid = i <= g.ni[0];
  } else {  // [j][i], pitch px
    k = sd ? g.ni[2] : 1;
    j = (int)(t / g.px) + 1;
    i = (int)(t % g.px) + 1;
    valid = i <= g.ni[0];
  }
}

template <typename T, int DIM>
__global__ void k_face_lift(Geom g, Weights w, const T* __restrict__ Q, T* __restrict__ Lx, T* __restrict__ Ly,
                            T* __restrict__ Lz, long long px_plane, long long py_plane, long long pz_plane) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  Q += b_ * g.nq;
  Lx += b_ * 2 * px_plane;
  Ly += b_ * 2 * py_plane;
  if (Lz) Lz += b_ * 2 * pz_plane;
  const long long tot = 2 * (px_plane + py_plane + (DIM == 3 ? pz_plane : 0));
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < tot;
       e += (long long)gridDim.x * blockDim.x) {
    int f;
    long long t;
    T* out;
    if (e < 2 * px_plane) {
      f = (int)(e / px_plane);
      t = e - f * px_plane;
      out = Lx + e;
    } else if (e < 2 * (px_plane + py_plane)) {
      const long long r = e - 2 * px_plane;
      f = 2 + (int)(r / py_plane);
      t = r - (f - 2) * py_plane;
      out = Ly + r;
    } else {
      const long long r = e - 2 * (px_plane + py_plane);
      f = 4 + (int)(r / pz_plane);
      t = r - (f - 4) * pz_plane;
      out = Lz + r;
    }
    int i, j, k, valid;
    face_node<DIM>(g, f, t, i, j, k, valid);
    T acc = 0;
    if (valid) {
      const int ax = f >> 1;
      const int dn = (f & 1) ? 1 : -1;  // offset of the face plane from the node
      for (int d1 = -1; d1 <= 1; ++d1)
        for (int d2 = (DIM == 3 ? -1 : 0); d2 <= (DIM == 3 ? 1 : 0); ++d2) {
          // tangential offsets: 3-D (d1, d2) along the two other axes; 2-D d1 only
          int dx = 0, dy = 0, dz = 0;
          if (ax == 0) { dx = dn; dy = d1; dz = d2; }
          else if (ax == 1) { dy = dn; dx = d1; dz = d2; }
          else { dz = dn; dx = d1; dy = d2; }
          const double wt = lw<DIM>(w, dx, dy, dz);
          if (wt == 0.0) continue;
          const int qi = i + dx, qj = j + dy, qk = k + dz;
          if (nbnd<DIM>(g, qi, qj, qk) == 1) acc += (T)wt * Q[qidx<DIM>(g, qi, qj, qk)];
        }
    }
    *out = acc;
  }
}

// 2-D: the V-solve's lift layers (couplings w0 across the face and wt to its two neighbours
// along it) and the U-solve's m1 Q_b / alpha_b, of every instance, in one pass over the lines
// of both axes.  Rows [2][n_y'] of the x faces, then [2][px] of the y faces (padding zero).
template <typename T>
__global__ void k_face_lifts2(Geom g, T w0x, T w0y, T wt, T m1, const T* __restrict__ Q, const T* __restrict__ ia,
                              T* __restrict__ Lx, T* __restrict__ Ly, T* __restrict__ Ux, T* __restrict__ Uy) {
  const long long b_ = blockIdx.y;
  Q += b_ * g.nq;
  ia += b_ * g.nnodal;
  const int nx = 2 * g.ni[1], tot = nx + 2 * g.px;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < tot; e += gridDim.x * blockDim.x) {
    const bool xf = e < nx;
    const int r = xf ? e : e - nx, len = xf ? g.ni[1] : g.px, n = xf ? g.ni[1] : g.ni[0];
    const int sd = r >= len, t = r - sd * len;  // face side, position along it (from 0)
    T l = 0, u = 0;
    if (t < n) {
      const T* q = Q + g.face_off[(xf ? 0 : 2) + sd];
      l = (xf ? w0x : w0y) * q[t];
      if (t > 0) l += wt * q[t - 1];
      if (t + 1 < n) l += wt * q[t + 1];
      const int i = xf ? (sd ? g.n[0] : 0) : t + 1, j = xf ? t + 1 : (sd ? g.n[1] : 0);
      u = m1 * q[t] * ia[(long long)j * g.nn[0] + i];
    }
    (xf ? Lx : Ly)[b_ * 2 * len + r] = l;
    (xf ? Ux : Uy)[b_ * 2 * len + r] = u;
  }
}

// out[q] = s * nodal(boundary node of q), a nodal field in Q's layout
template <typename T, int DIM>
__global__ void k_nodal_to_q(Geom g, T s, const T* __restrict__ nodal, T* __restrict__ out) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  nodal += b_ * g.nnodal;
  out += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    out[q] = s * nodal[nod(g, i, j, k)];
  }
}

// Both face-layer sets of the 3-D homogeneous matvec in one pass over Q, by 32 x 32 tiles of
// each face in Q's own layout (rows along the face's slower tangential axis, the faster one
// contiguous):
//   V-solve lift  Lf = w0 Q + w_fast (Q(s, f-1) + Q(s, f+1)) + w_slow (Q(s-1, f) + Q(s+1, f)),
//                 the 19-point operator's couplings of a layer node to the face (face normal
//                 weight w0, edge weights to the tangential neighbours; Q = 0 past the face's
//                 interior)
//   U-solve layer Uf = (m1 / alpha_b) Q, the factor from the nodal alpha in Q's layout (mq)
// The tile (with a one-node halo) is read coalesced into LDS; each output is written in its
// own layout -- along the same axis as Q for the y/z-face V layers and the z-face U layer,
// transposed (through LDS) for the x faces and the y-face U layer.  Layouts of face_lift, except
// the U-solve's y faces: [side][i][k] with k fastest (pitch n_z', no padding), the order in which
// the slowest-axis pass reads them.
template <typename T>
__global__ void __launch_bounds__(256) k_face_lifts3(Geom g, const T* __restrict__ Q, const T* __restrict__ mq,
                                                      FaceLiftW<T> lw, T* __restrict__ Lx, T* __restrict__ Ly,
                                                      T* __restrict__ Lz, T* __restrict__ Ux, T* __restrict__ Uy,
                                                      T* __restrict__ Uz) {
  constexpr int TS = 32;
  __shared__ T qt[TS + 2][TS + 3];
  __shared__ T vt[TS][TS + 1];
  __shared__ T ut[TS][TS + 1];
  // work-group -> (face, slow tile, fast tile)
  int b = blockIdx.x, f = 0;
  int nf = 0, ns = 0, tf = 0, ts = 0;
  for (f = 0; f < 6; ++f) {
    const int a = f >> 1;
    nf = a == 0 ? g.ni[1] : g.ni[0];  // faster tangential axis: y for x faces, x otherwise
    ns = a == 2 ? g.ni[1] : g.ni[2];  // slower: z for x and y faces, y for z faces
    tf = (nf + TS - 1) / TS;
    ts = (ns + TS - 1) / TS;
    if (b < tf * ts) break;
    b -= tf * ts;
  }
  if (f >= 6) return;
  const int a = f >> 1, sd = f & 1;
  const int s0 = (b / tf) * TS, f0 = (b % tf) * TS;
  const T* Qf = Q + g.face_off[f];
  const T* Mf = mq + g.face_off[f];
  const int lx = threadIdx.x & 31, ly = threadIdx.x >> 5;  // 32 x 8
  // Q tile with halo, zero past the face interior
  for (int r = ly; r < TS + 2; r += 8)
    for (int c = lx; c < TS + 2; c += 32) {
      const int ss = s0 + r - 1, ff = f0 + c - 1;
      qt[r][c] = (ss >= 0 && ss < ns && ff >= 0 && ff < nf) ? Qf[(long long)ss * nf + ff] : T(0);
    }
  __syncthreads();
  const T w0 = lw.w0[a], wf = lw.wf[a], ws = lw.ws[a];
  for (int r = ly; r < TS; r += 8) {
    const int ss = s0 + r, ff = f0 + lx;
    T v = 0, u = 0;
    if (ss < ns && ff < nf) {
      const T q = qt[r + 1][lx + 1];
      v = w0 * q + wf * (qt[r + 1][lx] + qt[r + 1][lx + 2]) + ws * (qt[r][lx + 1] + qt[r + 2][lx + 1]);
      u = q * Mf[(long long)ss * nf + ff];
    }
    vt[r][lx] = v;
    ut[r][lx] = u;
  }
  __syncthreads();
  // along Q's axes: row ss (slower axis), column ff (faster), pitch px; the padding columns
  // (px - n_x' < 32, all in the last tile, whose entries there are zero) are written too
  auto direct = [&](T* out, const T (*tile)[TS + 1], long long pitch) {
    for (int r = ly; r < TS; r += 8) {
      const int ss = s0 + r, ff = f0 + lx;
      if (ss < ns && ff < pitch) out[(long long)ss * pitch + ff] = tile[r][lx];
    }
  };
  // transposed: row ff, column ss, pitch ns
  auto transposed = [&](T* out, const T (*tile)[TS + 1]) {
    for (int r = ly; r < TS; r += 8) {
      const int ff = f0 + r, ss = s0 + lx;
      if (ff < nf && ss < ns) out[(long long)ff * ns + ss] = tile[lx][r];
    }
  };
  if (a == 0) {  // x faces: [side][j][k]
    transposed(Lx + (long long)sd * g.ni[1] * g.ni[2], vt);
    transposed(Ux + (long long)sd * g.ni[1] * g.ni[2], ut);
  } else if (a == 1) {  // y faces: V [side][k][px], U [side][i][k]
    direct(Ly + (long long)sd * g.ni[2] * g.px, vt, g.px);
    transposed(Uy + (long long)sd * g.ni[0] * g.ni[2], ut);
  } else {  // z faces: [side][j][px]
    direct(Lz + (long long)sd * g.ni[1] * g.px, vt, g.px);
    direct(Uz + (long long)sd * g.ni[1] * g.px, ut, g.px);
  }
}

// out[e] = sum_{b < count} in[b * stride + e], e < n, in a fixed order
template <typename T>
__global__ void k_partial_sum(long long n, int count, long long stride, const T* __restrict__ in,
                              T* __restrict__ out) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    T acc = 0;
    for (int b = 0; b < count; ++b) acc += in[b * stride + e];
    out[e] = acc;
  }
}

// Boundary residual from the face sums S = 6 U1 - 3/2 U2 + 2/9 U3 (formed in spectral space):
//   R = alpha_b h^-2 S - Q - src_q
//   3-D: x faces S = Fx[s][(j-1) n_z' + (k-1)], y faces Fy[s][(k-1) px + (i-1)],
//        z faces Fz[s][(j-1) px + (i-1)];  2-D: Fx[s][j-1], Fy[s][i-1]
template <typename T, int DIM>
__global__ void k_gather_faces(Geom g, const T* __restrict__ Fx, const T* __restrict__ Fy,
                               const T* __restrict__ Fz, const T* __restrict__ Q, const T* __restrict__ af,
                               const T* __restrict__ srcq, double* __restrict__ R) {
  const long long px_plane = DIM == 3 ? (long long)g.ni[1] * g.ni[2] : g.ni[1];
  const long long py_plane = DIM == 3 ? (long long)g.px * g.ni[2] : g.px;
  const long long pz_plane = (long long)g.px * g.ni[1];
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  Fx += b_ * 2 * px_plane;
  Fy += b_ * 2 * py_plane;
  if (DIM == 3) Fz += b_ * 2 * pz_plane;
  Q += b_ * g.nq;
  af += b_ * g.nq;
  if (srcq) srcq += b_ * g.nq;
  R += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    const int sd = st > 0 ? 0 : 1;  // low face (step +1) -> 0
    T S;
    if (ax == 0) {
      const long long r = DIM == 3 ? (long long)(j - 1) * g.ni[2] + (k - 1) : (j - 1);
      S = Fx[sd * px_plane + r];
    } else if (ax == 1) {
      const long long r = DIM == 3 ? (long long)(k - 1) * g.px + (i - 1) : (i - 1);
      S = Fy[sd * py_plane + r];
    } else {
      S = Fz[sd * pz_plane + (long long)(j - 1) * g.px + (i - 1)];
    }
    const T ih2 = (T)(1.0 / (g.h[ax] * g.h[ax]));
    T r = af[q] * ih2 * S - Q[q];
    if (srcq) r -= srcq[q];
    R[q] = (double)r;
  }
}

// FP64 residual of the coupled system at the interior nodes:
//   r_v = src_v + L_h[V]            (V = interior V, Q on face interiors, 0 on edges)
//   r_u = src_u + M(V/alpha) - L_h[U]   (U = interior U, 0 on the boundary)
template <typename T, int DIM>
__global__ void k_resid_vol(Geom g, Weights w, const double* __restrict__ U, const double* __restrict__ V,
                            const double* __restrict__ Q, const double* __restrict__ ia,
                            const double* __restrict__ src_u, const double* __restrict__ src_v,
                            T* __restrict__ ru, T* __restrict__ rv) {
  // rows (j, k) across work-groups, x across threads (32-bit row decode)
  const int nrow_ = DIM == 3 ? g.ni[1] * g.ni[2] : g.ni[1];
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i0_ = threadIdx.x; i0_ < g.px; i0_ += blockDim.x) {
    const long long e = (long long)r_ * g.px + i0_;
    const int i = i0_ + 1, j = (DIM == 3 ? r_ % g.ni[1] : r_) + 1, k = DIM == 3 ? r_ / g.ni[1] + 1 : 0;
    if (i > g.ni[0]) {
      rv[e] = T(0);
      ru[e] = T(0);
      continue;
    }
    double lv = 0, lu = 0, mv = 0;
    const int zlo = DIM == 3 ? -1 : 0, zhi = DIM == 3 ? 1 : 0;
    for (int dz = zlo; dz <= zhi; ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const double wt = lw<DIM>(w, dx, dy, dz);
          const int nzo = (dx != 0) + (dy != 0) + (dz != 0);
          if (wt == 0.0 && nzo > 1) continue;  // outside both stencils (M also reads nzo <= 1)
          const int qi = i + dx, qj = j + dy, qk = k + dz;
          const int nb = nbnd<DIM>(g, qi, qj, qk);
          double vq = 0, uq = 0;
          if (nb == 0) {
            const long long qe = inr(g, qi, qj, DIM == 3 ? qk : 1);
            vq = V[qe];
            uq = U[qe];
          } else if (nb == 1) {
            vq = Q[qidx<DIM>(g, qi, qj, qk)];
          }
          lv += wt * vq;
          lu += wt * uq;
          if (nzo <= 1) mv += (nzo == 0 ? w.m0 : w.m1) * vq * ia[nod(g, qi, qj, qk)];
        }
    rv[e] = (T)(src_v[e] + lv);
    ru[e] = (T)((src_u ? src_u[e] : 0.0) + mv - lu);
  }
}

template <typename T, int DIM>
__global__ void k_resid_q(Geom g, Weights w, const double* __restrict__ U, const double* __restrict__ Q,
                          const double* __restrict__ af, const double* __restrict__ src_q,
                          T* __restrict__ rq) {
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    double u[3];
#pragma unroll
    for (int m = 1; m <= 3; ++m) {
      const int ui = i + (ax == 0 ? st * m : 0), uj = j + (ax == 1 ? st * m : 0),
                uk = k + (ax == 2 ? st * m : 0);
      u[m - 1] = U[inr(g, ui, uj, DIM == 3 ? uk : 1)];
    }
    const double ih2 = 1.0 / (g.h[ax] * g.h[ax]);
    const double G = af[q] * ih2 * (w.os[1] * u[0] + w.os[2] * u[1] + w.os[3] * u[2]);
    rq[q] = (T)((src_q ? src_q[q] : 0.0) + Q[q] - G);
  }
}

// ---------------------------------------------------------------------------------
// setup (FP64 inputs)

__global__ void k_inv_alpha(long long n, const double* __restrict__ alpha, double* __restrict__ ia64,
                            float* __restrict__ ia32, double* __restrict__ bmin) {
  __shared__ double red[TPB];
  double mn = 1e300;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    const double a = alpha[e];
    mn = fmin(mn, a);
    const double r = 1.0 / a;
    ia64[e] = r;
    if (ia32) ia32[e] = (float)r;
  }
  red[threadIdx.x] = mn;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) bmin[blockIdx.x] = red[0];
}

template <int DIM>
__global__ void k_face_alpha(Geom g, const double* __restrict__ alpha, double* __restrict__ af64,
                             float* __restrict__ af32) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  alpha += b_ * g.nnodal;
  af64 += b_ * g.nq;
  if (af32) af32 += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    const double a = alpha[nod(g, i, j, k)];
    af64[q] = a;
    if (af32) af32[q] = (float)a;
  }
}

// src_v = M f + (L_h contributions of the known edge/corner values V = alpha * lapgD)
// src_u = -(L_h contributions of U = g_D on the boundary)
template <int DIM>
__global__ void k_src_vol(Geom g, Weights w, const double* __restrict__ f, const double* __restrict__ alpha,
                          const double* __restrict__ gD, const double* __restrict__ lapgD,
                          double* __restrict__ src_v, double* __restrict__ src_u) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  f += b_ * g.nnodal;
  alpha += b_ * g.nnodal;
  if (gD) gD += b_ * g.nnodal;
  if (lapgD) lapgD += b_ * g.nnodal;
  src_v += b_ * g.nalloc;
  if (src_u) src_u += b_ * g.nalloc;
  // rows (j, k) across work-groups, x across threads (32-bit row decode)
  const int nrow_ = DIM == 3 ? g.ni[1] * g.ni[2] : g.ni[1];
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i0_ = threadIdx.x; i0_ < g.px; i0_ += blockDim.x) {
    const long long e = (long long)r_ * g.px + i0_;
    const int i = i0_ + 1, j = (DIM == 3 ? r_ % g.ni[1] : r_) + 1, k = DIM == 3 ? r_ / g.ni[1] + 1 : 0;
    if (i > g.ni[0]) {
      src_v[e] = 0.0;
      if (src_u) src_u[e] = 0.0;
      continue;
    }
    double mf = w.m0 * f[nod(g, i, j, k)];
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int s = -1; s <= 1; s += 2)
        mf += w.m1 * f[nod(g, i + (a == 0 ? s : 0), j + (a == 1 ? s : 0), k + (a == 2 ? s : 0))];
    double ev = 0, eu = 0;
    const int zlo = DIM == 3 ? -1 : 0, zhi = DIM == 3 ? 1 : 0;
    for (int dz = zlo; dz <= zhi; ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const double wt = lw<DIM>(w, dx, dy, dz);
          if (wt == 0.0) continue;
          const int qi = i + dx, qj = j + dy, qk = k + dz;
          const int nb = nbnd<DIM>(g, qi, qj, qk);
          if (nb == 0) continue;
          const long long qn = nod(g, qi, qj, qk);
          if (nb >= 2 && lapgD) ev += wt * alpha[qn] * lapgD[qn];
          if (gD) eu += wt * gD[qn];
        }
    src_v[e] = mf + ev;
    if (src_u) src_u[e] = -eu;
  }
}

// src_q = -alpha_b [ a_0 g_D / h^2 + (11/3) g_N / h + lapgD ]   (known part of the q-row)
template <int DIM>
__global__ void k_src_q(Geom g, Weights w, const double* __restrict__ alpha, const double* __restrict__ gD,
                        const double* __restrict__ gN, const double* __restrict__ lapgD,
                        double* __restrict__ src_q) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  alpha += b_ * g.nnodal;
  if (gD) gD += b_ * g.nnodal;
  if (gN) gN += b_ * g.nnodal;
  if (lapgD) lapgD += b_ * g.nnodal;
  src_q += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    const long long b = nod(g, i, j, k);
    const double h = g.h[ax];
    double t = 0;
    if (gD) t += w.os[0] * gD[b] / (h * h);
    if (gN) t += w.os_gn * gN[b] / h;
    if (lapgD) t += lapgD[b];
    src_q[q] = -alpha[b] * t;
  }
}

// The v-equation's operator with a variable shift c = beta / alpha (nodal), on the interior:
//   y = -L_h[V] + M(c V),  V = X at interior nodes and 0 on the boundary (2-D)
__global__ void k_vapply(Geom g, Weights w, const double* __restrict__ X, const double* __restrict__ c,
                         double* __restrict__ y) {
  for (int r_ = blockIdx.x; r_ < g.ni[1]; r_ += gridDim.x)
    for (int i0_ = threadIdx.x; i0_ < g.px; i0_ += blockDim.x) {
      const long long e = (long long)r_ * g.px + i0_;
      const int i = i0_ + 1, j = r_ + 1;
      if (i > g.ni[0]) {
        y[e] = 0.0;
        continue;
      }
      double lv = 0, mv = 0;
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx) {
          const bool in = i + dx >= 1 && i + dx <= g.ni[0] && j + dy >= 1 && j + dy <= g.ni[1];
          const double vq = in ? X[e + dy * g.px + dx] : 0.0;
          lv += lw<2>(w, dx, dy, 0) * vq;
          if (dx == 0 || dy == 0) mv += (dx == 0 && dy == 0 ? w.m0 : w.m1) * c[(long long)(j + dy) * g.nn[0] + i + dx] * vq;
        }
      y[e] = mv - lv;
    }
}

// The same operator in 3-D, tiled: a work-group owns VTX x VTY columns and
// marches along z over kchunk planes, with the planes k-1, k, k+1 of its columns and their halo
// in LDS (zero on the boundary) and c X of plane k beside them, so every value is read from
// memory about once per plane instead of once per stencil point.  The next plane's values are on
// their way while a plane is summed: with loads waited for where they are stored, two trips to
// memory per plane were the time (128^3: 27.0 us, 20.8 now; 64.4 with chunks of 32 planes, 128
// work-groups).  part[b] and part[gridDim.x + b] are work-group b's parts of <u, y> and <y, y>: a
// sweep of its own over u and y took 10 us and a launch.
constexpr int VTX = 64, VTY = 8;
__global__ void __launch_bounds__(VTX * VTY) k_vapply_tile(Geom g, Weights w, const double* __restrict__ X,
                                                           const double* __restrict__ c, double* __restrict__ y,
                                                           int kchunk, const double* __restrict__ u,
                                                           double* __restrict__ part) {
  constexpr int HX = VTX + 2, HY = VTY + 2;
  __shared__ double xs[3][HY][HX];
  __shared__ double cs[HY][HX];
  const int ni0 = g.ni[0], ni1 = g.ni[1], ni2 = g.ni[2];
  const int tx = (ni0 + VTX - 1) / VTX, ty = (ni1 + VTY - 1) / VTY, tz = (ni2 + kchunk - 1) / kchunk;
  long long t = blockIdx.x;
  if (t >= (long long)tx * ty * tz) return;
  const int bx = (int)(t % tx);
  t /= tx;
  const int by = (int)(t % ty), bz = (int)(t / ty);
  const int lx = threadIdx.x % VTX, ly = threadIdx.x / VTX;
  const int ib = 1 + bx * VTX, jb = 1 + by * VTY;  // first column of the tile
  const int i = ib + lx, j = jb + ly;
  const bool mine = i <= ni0 && j <= ni1;
  const int k0 = 1 + bz * kchunk, k1 = min(ni2, k0 + kchunk - 1);
  const long long npl = (long long)g.nn[1] * g.nn[0];
  // this thread's halo positions (hx, hy) -> nodes (ib - 1 + hx, jb - 1 + hy), clamped to the far
  // faces (positions beyond them feed only columns whose outputs are not written)
  constexpr int NH = (HX * HY + VTX * VTY - 1) / (VTX * VTY);
  const long long xpl = (long long)ni1 * g.px;
  long long xoff[NH], coff[NH];
  bool xin[NH], used[NH];
#pragma unroll
  for (int q = 0; q < NH; ++q) {
    const int h = threadIdx.x + q * VTX * VTY;
    used[q] = h < HX * HY;
    const int gi = min(ib - 1 + h % HX, ni0 + 1), gj = min(jb - 1 + h / HX, ni1 + 1);
    xin[q] = used[q] && gi >= 1 && gi <= ni0 && gj >= 1 && gj <= ni1;
    xoff[q] = xin[q] ? (long long)(gj - 1) * g.px + (gi - 1) : 0;
    coff[q] = used[q] ? (long long)gj * g.nn[0] + gi : 0;
  }
  auto xval = [&](int q, int kk) { return xin[q] && kk >= 1 && kk <= ni2 ? X[(kk - 1) * xpl + xoff[q]] : 0.0; };
  double* const csf = &cs[0][0];
  double duy = 0, dyy = 0;
  int s0 = 0, s1 = 1, s2 = 2;  // slots of planes k-1, k, k+1
  const long long cown = mine ? (long long)j * g.nn[0] + i : 0, yown = mine ? (long long)(j - 1) * g.px + (i - 1) : 0;
  double cm = c[(k0 - 1) * npl + cown], cp = c[(k0 + 1) * npl + cown], c1 = c[k0 * npl + cown];
  double un = u[(k0 - 1) * xpl + yown];
#pragma unroll
  for (int q = 0; q < NH; ++q) {
    const int h = threadIdx.x + q * VTX * VTY;
    const double a = xval(q, k0 - 1), b = xval(q, k0), d = xval(q, k0 + 1), cq = c[k0 * npl + coff[q]];
    if (used[q]) {
      (&xs[s0][0][0])[h] = a;
      (&xs[s1][0][0])[h] = b;
      (&xs[s2][0][0])[h] = d;
      csf[h] = cq * b;
    }
  }
  __syncthreads();
  for (int k = k0; k <= k1; ++k) {
    // the next plane's values on their way while this one is summed
    double xn[NH], cn[NH], cnext = 0, unext = 0;
    const bool more = k < k1;
    if (more) {
#pragma unroll
      for (int q = 0; q < NH; ++q) {
        xn[q] = xval(q, k + 2);
        cn[q] = c[(k + 1) * npl + coff[q]];
      }
      cnext = c[(k + 2) * npl + cown];
      unext = u[k * xpl + yown];
    }
    if (mine) {
      const int hx = lx + 1, hy = ly + 1;
      const double (*pm)[HX] = xs[s0];
      const double (*pc)[HX] = xs[s1];
      const double (*pp)[HX] = xs[s2];
      double lv = w.c0 * pc[hy][hx];
      lv += w.cf[0] * (pc[hy][hx - 1] + pc[hy][hx + 1]);
      lv += w.cf[1] * (pc[hy - 1][hx] + pc[hy + 1][hx]);
      lv += w.cf[2] * (pm[hy][hx] + pp[hy][hx]);
      lv += w.ce[0] * (pc[hy - 1][hx - 1] + pc[hy - 1][hx + 1] + pc[hy + 1][hx - 1] + pc[hy + 1][hx + 1]);
      lv += w.ce[1] * (pm[hy][hx - 1] + pm[hy][hx + 1] + pp[hy][hx - 1] + pp[hy][hx + 1]);
      lv += w.ce[2] * (pm[hy - 1][hx] + pm[hy + 1][hx] + pp[hy - 1][hx] + pp[hy + 1][hx]);
      double mv = w.m0 * cs[hy][hx] + w.m1 * (cs[hy][hx - 1] + cs[hy][hx + 1] + cs[hy - 1][hx] + cs[hy + 1][hx]);
      mv += w.m1 * (cm * pm[hy][hx] + cp * pp[hy][hx]);
      const double out = mv - lv;
      y[(k - 1) * xpl + yown] = out;
      duy += un * out;
      dyy += out * out;
    }
    if (more) {
      __syncthreads();  // slot s0 (plane k-1) and cs no longer read
#pragma unroll
      for (int q = 0; q < NH; ++q) {
        const int h = threadIdx.x + q * VTX * VTY;
        if (used[q]) {
          (&xs[s0][0][0])[h] = xn[q];
          csf[h] = cn[q] * (&xs[s2][0][0])[h];
        }
      }
      cm = c1;
      c1 = cp;
      cp = cnext;
      un = unext;
      const int tmp = s0;
      s0 = s1;
      s1 = s2;
      s2 = tmp;
      __syncthreads();
    }
  }
  __shared__ double red[2][VTX * VTY / 64];
  for (int m = 32; m >= 1; m >>= 1) {
    duy += __shfl_xor(duy, m, 64);
    dyy += __shfl_xor(dyy, m, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = duy;
    red[1][threadIdx.x >> 6] = dyy;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double r = red[threadIdx.x][0];
    for (int q = 1; q < VTX * VTY / 64; ++q) r += red[threadIdx.x][q];
    part[(long long)threadIdx.x * gridDim.x + blockIdx.x] = r;
  }
}

// The V-solve's start from V = 0 inside: r = rh = p = src - A V with V = Q on the face interiors
// (src may be null), and part[b], work-group b's part of <r, r>.  Only the layer next to the
// boundary has stencils to sum; the rest is a sweep over the vectors.  128^3: 79 us for the
// general stencil over zeros and 30 for the sweeps after it, 29 here.
template <int DIM>
__global__ void __launch_bounds__(TPB)
    k_vstart(Geom g, Weights w, long long n, const double* __restrict__ Q, const double* __restrict__ c,
             const double* __restrict__ src, double* __restrict__ r, double* __restrict__ rh,
             double* __restrict__ p, double* __restrict__ part) {
  __shared__ double red[TPB / 64];
  double rr = 0;
  for (long long e = blockIdx.x * (long long)TPB + threadIdx.x; e < n; e += (long long)gridDim.x * TPB) {
    const long long row = e / g.px;
    const int i = (int)(e - row * g.px) + 1;
    const int k = DIM == 3 ? (int)(row / g.ni[1]) + 1 : 0;
    const int j = (int)(row - (DIM == 3 ? (long long)(k - 1) * g.ni[1] : 0)) + 1;
    double v = 0;
    if (i <= g.ni[0]) {
      double lv = 0, mv = 0;
      const int pos[3] = {i, j, k};
#pragma unroll
      for (int f = 0; f < 2 * DIM; ++f) {
        const int ax = f >> 1, sd = f & 1 ? 1 : -1;
        if (pos[ax] != (sd > 0 ? g.ni[ax] : 1)) continue;
#pragma unroll
        for (int o = 0; o < 2 * DIM - 1; ++o) {  // the node in the face, and its neighbours there
          int d[3] = {0, 0, 0};
          d[ax] = sd;
          if (o) {
            const int b = (o - 1) >> 1, tr = b < ax ? b : b + 1;
            d[tr] = (o - 1) & 1 ? 1 : -1;
            if (pos[tr] + d[tr] < 1 || pos[tr] + d[tr] > g.ni[tr]) continue;  // edges and corners are zero
          }
          const double vq = Q[qidx<DIM>(g, i + d[0], j + d[1], k + d[2])];
          lv += lw<DIM>(w, d[0], d[1], d[2]) * vq;
          if (!o) mv += w.m1 * c[nod(g, i + d[0], j + d[1], k + d[2])] * vq;
        }
      }
      v = (src ? src[e] : 0.0) + lv - mv;
    }
    r[e] = v;
    rh[e] = v;
    p[e] = v;
    rr += v * v;
  }
  for (int m = 32; m >= 1; m >>= 1) rr += __shfl_xor(rr, m, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = rr;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < TPB / 64; ++q) rr += red[q];
    part[blockIdx.x] = rr;
  }
}

// per-block minimum and maximum of x: part[2 b] = min, part[2 b + 1] = max
__global__ void k_minmax(long long n, const double* __restrict__ x, double* __restrict__ part) {
  __shared__ double rmin[TPB], rmax[TPB];
  double mn = 1e300, mx = -1e300;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    mn = fmin(mn, x[e]);
    mx = fmax(mx, x[e]);
  }
  rmin[threadIdx.x] = mn;
  rmax[threadIdx.x] = mx;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      rmin[threadIdx.x] = fmin(rmin[threadIdx.x], rmin[threadIdx.x + s]);
      rmax[threadIdx.x] = fmax(rmax[threadIdx.x], rmax[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = rmin[0];
    part[2 * blockIdx.x + 1] = rmax[0];
  }
}

// Navier faces (bit f of `mask`, f = 2 axis + side): Delta u = g_L is given there, so V =
// alpha g_L is known and the face's q-rows read R = alpha g_L - Q.  The gather's one-sided
// term is switched off (af = 0) and the known part becomes src_q = -alpha g_L.
template <int DIM>
__global__ void k_navier(Geom g, int mask, const double* __restrict__ alpha, const double* __restrict__ gL,
                         double* __restrict__ af64, float* __restrict__ af32, double* __restrict__ src_q) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  alpha += b_ * g.nnodal;
  if (gL) gL += b_ * g.nnodal;
  af64 += b_ * g.nq;
  if (af32) af32 += b_ * g.nq;
  src_q += b_ * g.nq;
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    const int f = 2 * ax + (st > 0 ? 0 : 1);  // low face (step +1) -> side 0
    if (!((mask >> f) & 1)) continue;
    const long long b = nod(g, i, j, k);
    af64[q] = 0.0;
    if (af32) af32[q] = 0.0f;
    src_q[q] = gL ? -alpha[b] * gL[b] : 0.0;
  }
}

// ---------------------------------------------------------------------------------
// Triharmonic extension (Sec. 4.2): Delta u = v, Delta v = w, Delta w = f, each by the
// compact scheme L_h X = M rhs, with w = Q on the face interiors (a Navier face's q-rows fix
// Q to Delta^2 u there).  The Schur matvec chains three Dirichlet solves (W from Q, V from W,
// U from V) and closes with the q-row of a clamped face,
//   R = h^-4 (a_1 U_1 + a_2 U_2 + a_3 U_3 + a_4 U_4) + (data) - Q,
// the one-sided fourth normal derivative that uses u, u_n, u_nn and the four nearest
// interior nodes: its weights solve the Taylor moment conditions through degree 6, i.e.
// h^4 d4u = a_0 u_0 + sum_k a_k U_k + c_1 h du + c_2 h^2 d2u + O(h^7) along the inward normal
// (du, d2u, d4u its derivatives) with a = (11669/144, -104, 57/2, -56/9, 11/16),
// c_1 = 755/12, c_2 = 35/2.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ double tri_a(int k) {
  return k == 1 ? -104.0 : (k == 2 ? 57.0 / 2.0 : (k == 3 ? -56.0 / 9.0 : 11.0 / 16.0));
}

// Interior sources of the three solves (known boundary values moved to the right-hand side):
//   sw = L_h[W on edges and corners] - M f     (the W-solve as W = -L^-1(sw + L_h^bnd[Q]))
//   sv = -L_h[V on the boundary]               (V = L^-1(M W + sv), W = Q on face interiors)
//   su = M[V on face interiors] - L_h[g_D]     (U = L^-1(M V + su))
// with V = lapu (Delta u) on every boundary node and W = bilap on edges and corners.
template <int DIM>
__global__ void k_tri_src(Geom g, Weights w, const double* __restrict__ f, const double* __restrict__ gD,
                          const double* __restrict__ lapu, const double* __restrict__ bilap,
                          double* __restrict__ sw, double* __restrict__ sv, double* __restrict__ su) {
  const int nrow_ = DIM == 3 ? g.ni[1] * g.ni[2] : g.ni[1];
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i0_ = threadIdx.x; i0_ < g.px; i0_ += blockDim.x) {
    const long long e = (long long)r_ * g.px + i0_;
    const int i = i0_ + 1, j = (DIM == 3 ? r_ % g.ni[1] : r_) + 1, k = DIM == 3 ? r_ / g.ni[1] + 1 : 0;
    if (i > g.ni[0]) {
      sw[e] = sv[e] = su[e] = 0.0;
      continue;
    }
    double mf = f ? w.m0 * f[nod(g, i, j, k)] : 0.0, mv = 0.0;
#pragma unroll
    for (int a = 0; a < DIM; ++a)
#pragma unroll
      for (int s = -1; s <= 1; s += 2) {
        const int qi = i + (a == 0 ? s : 0), qj = j + (a == 1 ? s : 0), qk = k + (a == 2 ? s : 0);
        const long long qn = nod(g, qi, qj, qk);
        if (f) mf += w.m1 * f[qn];
        if (lapu && nbnd<DIM>(g, qi, qj, qk) == 1) mv += w.m1 * lapu[qn];
      }
    double lw_ = 0, lv = 0, lu = 0;
    const int zlo = DIM == 3 ? -1 : 0, zhi = DIM == 3 ? 1 : 0;
    for (int dz = zlo; dz <= zhi; ++dz)
      for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
          const double wt = lw<DIM>(w, dx, dy, dz);
          if (wt == 0.0) continue;
          const int qi = i + dx, qj = j + dy, qk = k + dz;
          const int nb = nbnd<DIM>(g, qi, qj, qk);
          if (nb == 0) continue;
          const long long qn = nod(g, qi, qj, qk);
          if (nb >= 2 && bilap) lw_ += wt * bilap[qn];
          if (lapu) lv += wt * lapu[qn];
          if (gD) lu += wt * gD[qn];
        }
    sw[e] = lw_ - mf;
    sv[e] = -lv;
    su[e] = mv - lu;
  }
}

// Known part of the q-rows and the face coefficient: on a clamped face
//   src_q = -[ h^-4 (a_0 g_D - c_1 h g_N + c_2 h^2 g_NN) + tang4 ]   (g_N outward = -du),
//   af = 1;  on a Navier face (bit 2 axis + side of mask) src_q = -bilap, af = 0.
template <int DIM>
__global__ void k_tri_srcq(Geom g, int mask, const double* __restrict__ gD, const double* __restrict__ gN,
                           const double* __restrict__ gNN, const double* __restrict__ tang4,
                           const double* __restrict__ bilap, double* __restrict__ src_q, double* __restrict__ af64,
                           float* __restrict__ af32) {
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    const int f = 2 * ax + (st > 0 ? 0 : 1);
    const long long b = nod(g, i, j, k);
    double sq, a;
    if ((mask >> f) & 1) {
      sq = bilap ? -bilap[b] : 0.0;
      a = 0.0;
    } else {
      const double h = g.h[ax];
      double t = 0;
      if (gD) t += (11669.0 / 144.0) * gD[b];
      if (gN) t -= (755.0 / 12.0) * h * gN[b];
      if (gNN) t += (35.0 / 2.0) * h * h * gNN[b];
      t /= h * h * h * h;
      if (tang4) t += tang4[b];
      sq = -t;
      a = 1.0;
    }
    src_q[q] = sq;
    af64[q] = a;
    if (af32) af32[q] = (float)a;
  }
}

// R = af h^-4 sum_{k=1..4} a_k U_k - Q - src_q at every face-interior node
template <typename T, int DIM>
__global__ void k_gather_tri(Geom g, const T* __restrict__ U, const T* __restrict__ Q, const T* __restrict__ af,
                             const T* __restrict__ srcq, double* __restrict__ R) {
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < g.nq; q += gridDim.x * blockDim.x) {
    int i, j, k, ax, st;
    dec_q<DIM>(g, q, i, j, k, ax, st);
    T acc = 0;
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
      const int ui = i + (ax == 0 ? st * m : 0), uj = j + (ax == 1 ? st * m : 0), uk = k + (ax == 2 ? st * m : 0);
      acc += (T)tri_a(m) * U[inr(g, ui, uj, DIM == 3 ? uk : 1)];
    }
    const double h = g.h[ax];
    T r = af[q] * (T)(1.0 / (h * h * h * h)) * acc - Q[q];
    if (srcq) r -= srcq[q];
    R[q] = (double)r;
  }
}

// nodal outputs
template <typename T, int DIM>
__global__ void k_out_u(Geom g, const T* __restrict__ Ui, const double* __restrict__ gD, double* __restrict__ u) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  Ui += b_ * g.nalloc;
  if (gD) gD += b_ * g.nnodal;
  u += b_ * g.nnodal;
  // nodal rows (j, k) across work-groups, x across threads
  const int nrow_ = g.nn[1] * (DIM == 3 ? g.nn[2] : 1);
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i = threadIdx.x; i < g.nn[0]; i += blockDim.x) {
    const long long e = (long long)r_ * g.nn[0] + i;
    const int j = r_ % g.nn[1];
    const int k = r_ / g.nn[1];
    const int nb = nbnd<DIM>(g, i, j, k);
    u[e] = nb == 0 ? (double)Ui[inr(g, i, j, DIM == 3 ? k : 1)] : (gD ? gD[e] : 0.0);
  }
}

template <typename T, int DIM>
__global__ void k_out_v(Geom g, const T* __restrict__ Vi, const double* __restrict__ Q,
                        const double* __restrict__ vedge, double* __restrict__ v) {
  const long long b_ = blockIdx.y;  // instance of a batch (gridDim.y = g.nb)
  Vi += b_ * g.nalloc;
  Q += b_ * g.nq;
  if (vedge) vedge += b_ * g.nnodal;
  v += b_ * g.nnodal;
  // nodal rows (j, k) across work-groups, x across threads
  const int nrow_ = g.nn[1] * (DIM == 3 ? g.nn[2] : 1);
  for (int r_ = blockIdx.x; r_ < nrow_; r_ += gridDim.x)
  for (int i = threadIdx.x; i < g.nn[0]; i += blockDim.x) {
    const long long e = (long long)r_ * g.nn[0] + i;
    const int j = r_ % g.nn[1];
    const int k = r_ / g.nn[1];
    const int nb = nbnd<DIM>(g, i, j, k);
    double val;
    if (nb == 0) val = (double)Vi[inr(g, i, j, DIM == 3 ? k : 1)];
    else if (nb == 1) val = Q[qidx<DIM>(g, i, j, k)];
    else val = vedge ? vedge[e] : 0.0;
    v[e] = val;
  }
}

template <typename Ti, typename To>
__global__ void k_cvt(long long n, const Ti* __restrict__ in, To* __restrict__ out) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    out[e] = (To)in[e];
}

template <typename Tx>
__global__ void k_acc(long long n, const Tx* __restrict__ x, double* __restrict__ y) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    y[e] += (double)x[e];
}

template <typename Tx>
__global__ void k_absmax(long long n, const Tx* __restrict__ x, double* __restrict__ bmax) {
  __shared__ double red[TPB];
  double m = 0;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    m = fmax(m, fabs((double)x[e]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) bmax[blockIdx.x] = red[0];
}

// rows x cols block copy between arrays with different row pitches (with conversion); columns
// from cols to wide are written as zeros
template <typename Ti, typename To>
__global__ void k_pitch_copy(long long rows, int cols, int wide, const Ti* __restrict__ in, long long ip,
                             To* __restrict__ out, long long op) {
  const long long n = rows * wide;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    const long long r = e / wide;
    const int c = (int)(e - r * wide);
    out[r * op + c] = c < cols ? (To)in[r * ip + c] : To(0);
  }
}

__global__ void k_mul(long long n, const double* __restrict__ a, const double* __restrict__ b,
                      double* __restrict__ out) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    out[e] = a[e] * b[e];
}

__global__ void k_fill(long long n, double v, double* __restrict__ x) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x)
    x[e] = v;
}

}  // namespace

// ---------------------------------------------------------------------------------
// launchers

#define LAUNCH_DIM(KER, grid, ...)                                                     \
  do {                                                                                 \
    if (g.dim == 3) hipLaunchKernelGGL((KER<3>), grid, dim3(TPB), 0, st, __VA_ARGS__); \
    else hipLaunchKernelGGL((KER<2>), grid, dim3(TPB), 0, st, __VA_ARGS__);           \
    AHOC_HIP_TRY(hipGetLastError());                                                   \
  } while (0)

#define LAUNCH_TDIM(KER, T, grid, ...)                                                     \
  do {                                                                                     \
    if (g.dim == 3) hipLaunchKernelGGL((KER<T, 3>), grid, dim3(TPB), 0, st, __VA_ARGS__);  \
    else hipLaunchKernelGGL((KER<T, 2>), grid, dim3(TPB), 0, st, __VA_ARGS__);            \
    AHOC_HIP_TRY(hipGetLastError());                                                       \
  } while (0)

template <typename T>
int lift(const Geom& g, const Weights& w, const T* Q, const T* src, T* G, hipStream_t st) {
  LAUNCH_TDIM(k_lift, T, dim3(interior_rows(g), g.nb), g, w, Q, src, G);
  return ST_OK;
}

template <typename T>
int rhs_u(const Geom& g, const Weights& w, const T* V, const T* Q, const T* ia, const T* src, T* G,
          hipStream_t st) {
  if (g.dim == 3) {
    // chunks of 32 planes, shorter (the halo planes are 2 / kchunk more reads) until four
    // work-groups of 512 threads meet on every compute unit: at 128^3 chunks of 4 planes
    // (14 us; 128 work-groups of 32-plane chunks 121 us)
    const long long cols = (long long)((g.px + RBX - 1) / RBX) * ((g.ni[1] + RBY - 1) / RBY);
    const int kchunk = (int)std::max<long long>(4, std::min<long long>(32, cols * g.ni[2] / 1024));
    const long long total = cols * ((g.ni[2] + kchunk - 1) / kchunk);
    if (total > 0x3fffffffLL) return ST_UNSUPPORTED;
    hipLaunchKernelGGL((k_rhs_u_blk<T>), dim3(8u * (unsigned)((total + 7) / 8)), dim3(RBX * RBY), 0, st, g, w, V, Q,
                       ia, src, G, kchunk);
    AHOC_HIP_TRY(hipGetLastError());
    return ST_OK;
  }
  const int nrow = g.ni[1];
  LAUNCH_TDIM(k_rhs_u, T, dim3((unsigned)(nrow < 1 ? 1 : nrow), g.nb), g, w, V, Q, ia, src, G);
  return ST_OK;
}

template <typename T>
int gather(const Geom& g, const Weights& w, const T* U, const T* Q, const T* af, const T* srcq,
           double* R, hipStream_t st) {
  LAUNCH_TDIM(k_gather, T, dim3(nblocks(g.nq), g.nb), g, w, U, Q, af, srcq, R);
  return ST_OK;
}

template <typename T>
int face_lift(const Geom& g, const Weights& w, const T* Q, T* Lx, T* Ly, T* Lz, hipStream_t st) {
  const long long pxp = g.dim == 3 ? (long long)g.ni[1] * g.ni[2] : g.ni[1];
  const long long pyp = g.dim == 3 ? (long long)g.px * g.ni[2] : g.px;
  const long long pzp = g.dim == 3 ? (long long)g.px * g.ni[1] : 0;
  const long long tot = 2 * (pxp + pyp + pzp);
  LAUNCH_TDIM(k_face_lift, T, dim3(nblocks(tot), g.nb), g, w, Q, Lx, Ly, Lz, pxp, pyp, pzp);
  return ST_OK;
}

template <typename T>
int face_lifts3(const Geom& g, const Weights& wv, const T* Q, const T* mq, T* Lx, T* Ly, T* Lz, T* Ux, T* Uy,
                T* Uz, hipStream_t st) {
  if (g.dim != 3 || g.nb != 1 || g.px - g.ni[0] >= 32) return ST_UNSUPPORTED;
  // the V lift's couplings per face axis a: normal, then edge weights to the faster and the
  // slower tangential neighbour (xy = ce[0], xz = ce[1], yz = ce[2])
  FaceLiftW<T> lw;
  lw.w0[0] = (T)wv.cf[0];
  lw.wf[0] = (T)wv.ce[0];
  lw.ws[0] = (T)wv.ce[1];
  lw.w0[1] = (T)wv.cf[1];
  lw.wf[1] = (T)wv.ce[0];
  lw.ws[1] = (T)wv.ce[2];
  lw.w0[2] = (T)wv.cf[2];
  lw.wf[2] = (T)wv.ce[1];
  lw.ws[2] = (T)wv.ce[2];
  long long blocks = 0;
  for (int f = 0; f < 6; ++f) {
    const int a = f >> 1;
    const int nf = a == 0 ? g.ni[1] : g.ni[0], ns = a == 2 ? g.ni[1] : g.ni[2];
    blocks += (long long)((nf + 31) / 32) * ((ns + 31) / 32);
  }
  if (blocks <= 0) return ST_OK;
  if (blocks > 0x7fffffffLL) return ST_UNSUPPORTED;
  hipLaunchKernelGGL((k_face_lifts3<T>), dim3((unsigned)blocks), dim3(256), 0, st, g, Q, mq, lw, Lx, Ly, Lz, Ux,
                     Uy, Uz);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename T>
int face_lifts2(const Geom& g, const Weights& wv, const T* Q, const T* ia, T* Lx, T* Ly, T* Ux, T* Uy, hipStream_t st) {
  if (g.dim != 2) return ST_UNSUPPORTED;
  hipLaunchKernelGGL((k_face_lifts2<T>), dim3(nblocks(2LL * (g.ni[1] + g.px)), g.nb), dim3(TPB), 0, st, g, (T)wv.cf[0],
                     (T)wv.cf[1], (T)wv.ce[0], (T)wv.m1, Q, ia, Lx, Ly, Ux, Uy);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename T>
int nodal_to_q(const Geom& g, double s, const T* nodal, T* out, hipStream_t st) {
  LAUNCH_TDIM(k_nodal_to_q, T, dim3(nblocks(g.nq), g.nb), g, (T)s, nodal, out);
  return ST_OK;
}

template <typename T>
int partial_sum(long long n, int count, long long stride, const T* in, T* out, hipStream_t st) {
  hipLaunchKernelGGL((k_partial_sum<T>), dim3(nblocks(n)), dim3(TPB), 0, st, n, count, stride, in, out);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename T>
int gather_faces(const Geom& g, const T* Fx, const T* Fy, const T* Fz, const T* Q, const T* af,
                 const T* srcq, double* R, hipStream_t st) {
  LAUNCH_TDIM(k_gather_faces, T, dim3(nblocks(g.nq), g.nb), g, Fx, Fy, Fz, Q, af, srcq, R);
  return ST_OK;
}

template <typename T>
int resid64(const Geom& g, const Weights& w, const double* U, const double* V, const double* Q,
            const double* ia, const double* af, const double* src_u, const double* src_v,
            const double* src_q, T* ru, T* rv, T* rq, hipStream_t st) {
  LAUNCH_TDIM(k_resid_vol, T, dim3(interior_rows(g)), g, w, U, V, Q, ia, src_u, src_v, ru, rv);
  LAUNCH_TDIM(k_resid_q, T, dim3(nblocks(g.nq)), g, w, U, Q, af, src_q, rq);
  return ST_OK;
}

int setup_inv_alpha(long long n, const double* alpha, double* ia64, float* ia32, double* bmin,
                    int nb, hipStream_t st) {
  hipLaunchKernelGGL(k_inv_alpha, dim3(nb), dim3(TPB), 0, st, n, alpha, ia64, ia32, bmin);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int setup_face_alpha(const Geom& g, const double* alpha, double* af64, float* af32, hipStream_t st) {
  LAUNCH_DIM(k_face_alpha, dim3(nblocks(g.nq), g.nb), g, alpha, af64, af32);
  return ST_OK;
}

namespace {
// Tiles of k_vapply_tile: chunks of 32 planes, shorter until two work-groups of 512 threads meet
// on every compute unit.
long long vapply_tiles(const Geom& g, int* kchunk) {
  const long long cols = (long long)((g.ni[0] + VTX - 1) / VTX) * ((g.ni[1] + VTY - 1) / VTY);
  *kchunk = (int)std::max<long long>(4, std::min<long long>(32, cols * g.ni[2] / 512));
  return cols * ((g.ni[2] + *kchunk - 1) / *kchunk);
}
}  // namespace

int vapply_dot_blocks(const Geom& g) {
  int kchunk;
  return g.dim == 3 && g.nb == 1 ? (int)std::min<long long>(vapply_tiles(g, &kchunk), 1 << 30) : 0;
}

int vapply_dot(const Geom& g, const Weights& w, const double* X, const double* c, double* y, const double* u,
               double* part, hipStream_t st) {
  if (g.nb != 1 || g.dim != 3) return ST_UNSUPPORTED;
  // (the row padding of y is never written: the callers' output arrays keep it zero)
  int kchunk;
  const long long tiles = vapply_tiles(g, &kchunk);
  hipLaunchKernelGGL(k_vapply_tile, dim3((unsigned)tiles), dim3(VTX * VTY), 0, st, g, w, X, c, y, kchunk, u, part);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int vapply(const Geom& g, const Weights& w, const double* X, const double* c, double* y, hipStream_t st) {
  if (g.nb != 1 || g.dim != 2) return ST_UNSUPPORTED;
  hipLaunchKernelGGL(k_vapply, dim3(interior_rows(g)), dim3(TPB), 0, st, g, w, X, c, y);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int vstart(const Geom& g, const Weights& w, long long n, const double* Q, const double* c, const double* src, double* r,
           double* rh, double* p, double* part, int nb, hipStream_t st) {
  if (g.nb != 1) return ST_UNSUPPORTED;
  LAUNCH_DIM(k_vstart, dim3(nb), g, w, n, Q, c, src, r, rh, p, part);
  return ST_OK;
}

int minmax_partial(long long n, const double* x, double* part, int nblocks, hipStream_t st) {
  hipLaunchKernelGGL(k_minmax, dim3(nblocks), dim3(TPB), 0, st, n, x, part);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int setup_navier(const Geom& g, int mask, const double* alpha, const double* gL, double* af64, float* af32,
                 double* src_q, hipStream_t st) {
  LAUNCH_DIM(k_navier, dim3(nblocks(g.nq), g.nb), g, mask, alpha, gL, af64, af32, src_q);
  return ST_OK;
}

int tri_sources(const Geom& g, const Weights& w, const double* f, const double* gD, const double* lapu,
                const double* bilap, double* sw, double* sv, double* su, hipStream_t st) {
  if (g.nb != 1) return ST_INVALID;
  LAUNCH_DIM(k_tri_src, dim3(interior_rows(g)), g, w, f, gD, lapu, bilap, sw, sv, su);
  return ST_OK;
}

int tri_srcq(const Geom& g, int mask, const double* gD, const double* gN, const double* gNN, const double* tang4,
             const double* bilap, double* src_q, double* af64, float* af32, hipStream_t st) {
  if (g.nb != 1) return ST_INVALID;
  LAUNCH_DIM(k_tri_srcq, dim3(nblocks(g.nq)), g, mask, gD, gN, gNN, tang4, bilap, src_q, af64, af32);
  return ST_OK;
}

template <typename T>
int gather_tri(const Geom& g, const T* U, const T* Q, const T* af, const T* srcq, double* R, hipStream_t st) {
  if (g.nb != 1) return ST_INVALID;
  LAUNCH_TDIM(k_gather_tri, T, dim3(nblocks(g.nq)), g, U, Q, af, srcq, R);
  return ST_OK;
}
template int gather_tri<float>(const Geom&, const float*, const float*, const float*, const float*, double*,
                               hipStream_t);
template int gather_tri<double>(const Geom&, const double*, const double*, const double*, const double*, double*,
                                hipStream_t);

int setup_sources(const Geom& g, const Weights& w, const double* f, const double* alpha,
                  const double* gD, const double* gN, const double* lapgD, double* src_v,
                  double* src_u, double* src_q, hipStream_t st) {
  LAUNCH_DIM(k_src_vol, dim3(interior_rows(g), g.nb), g, w, f, alpha, gD, lapgD, src_v, src_u);
  LAUNCH_DIM(k_src_q, dim3(nblocks(g.nq), g.nb), g, w, alpha, gD, gN, lapgD, src_q);
  return ST_OK;
}

template <typename T>
int out_u(const Geom& g, const T* Ui, const double* gD, double* u, hipStream_t st) {
  LAUNCH_TDIM(k_out_u, T, dim3(nodal_rows(g), g.nb), g, Ui, gD, u);
  return ST_OK;
}

template <typename T>
int out_v(const Geom& g, const T* Vi, const double* Q, const double* vedge, double* v, hipStream_t st) {
  LAUNCH_TDIM(k_out_v, T, dim3(nodal_rows(g), g.nb), g, Vi, Q, vedge, v);
  return ST_OK;
}

template <typename Ti, typename To>
int pitch_copy(long long rows, int cols, const Ti* in, long long ip, To* out, long long op, hipStream_t st, int wide) {
  if (wide < cols) wide = cols;
  hipLaunchKernelGGL((k_pitch_copy<Ti, To>), dim3(nblocks(rows * wide)), dim3(TPB), 0, st, rows, cols, wide, in, ip, out,
                     op);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int mul(long long n, const double* a, const double* b, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_mul, dim3(nblocks(n)), dim3(TPB), 0, st, n, a, b, out);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename Ti, typename To>
int convert(long long n, const Ti* in, To* out, hipStream_t st) {
  hipLaunchKernelGGL((k_cvt<Ti, To>), dim3(nblocks(n)), dim3(TPB), 0, st, n, in, out);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename Tx> int accumulate(long long n, const Tx* x, double* y, hipStream_t st) {
  hipLaunchKernelGGL((k_acc<Tx>), dim3(nblocks(n)), dim3(TPB), 0, st, n, x, y);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

template <typename Tx>
int absmax_partial(long long n, const Tx* x, double* bmax, int nb, hipStream_t st) {
  hipLaunchKernelGGL((k_absmax<Tx>), dim3(nb), dim3(TPB), 0, st, n, x, bmax);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

int fill(long long n, double v, double* x, hipStream_t st) {
  hipLaunchKernelGGL(k_fill, dim3(nblocks(n)), dim3(TPB), 0, st, n, v, x);
  AHOC_HIP_TRY(hipGetLastError());
  return ST_OK;
}

#define INST_T(T)                                                                                  \
  template int face_lift<T>(const Geom&, const Weights&, const T*, T*, T*, T*, hipStream_t);       \
  template int face_lifts2<T>(const Geom&, const Weights&, const T*, const T*, T*, T*, T*, T*, hipStream_t);   \
  template int face_lifts3<T>(const Geom&, const Weights&, const T*, const T*, T*, T*, T*, T*, T*, T*,        \
                              hipStream_t);                                                        \
  template int nodal_to_q<T>(const Geom&, double, const T*, T*, hipStream_t);                      \
  template int partial_sum<T>(long long, int, long long, const T*, T*, hipStream_t);               \
  template int gather_faces<T>(const Geom&, const T*, const T*, const T*, const T*, const T*,       \
                               const T*, double*, hipStream_t);                                    \
  template int lift<T>(const Geom&, const Weights&, const T*, const T*, T*, hipStream_t);         \
  template int rhs_u<T>(const Geom&, const Weights&, const T*, const T*, const T*, const T*, T*,   \
                        hipStream_t);                                                              \
  template int gather<T>(const Geom&, const Weights&, const T*, const T*, const T*, const T*,       \
                         double*, hipStream_t);                                                    \
  template int resid64<T>(const Geom&, const Weights&, const double*, const double*, const double*, \
                          const double*, const double*, const double*, const double*,              \
                          const double*, T*, T*, T*, hipStream_t);                                 \
  template int out_u<T>(const Geom&, const T*, const double*, double*, hipStream_t);               \
  template int out_v<T>(const Geom&, const T*, const double*, const double*, double*, hipStream_t); \
  template int accumulate<T>(long long, const T*, double*, hipStream_t);                           \
  template int absmax_partial<T>(long long, const T*, double*, int, hipStream_t);

INST_T(float)
INST_T(double)
template int pitch_copy<double, float>(long long, int, const double*, long long, float*, long long, hipStream_t, int);
template int pitch_copy<float, double>(long long, int, const float*, long long, double*, long long, hipStream_t, int);
template int pitch_copy<double, double>(long long, int, const double*, long long, double*, long long, hipStream_t, int);
template int convert<double, float>(long long, const double*, float*, hipStream_t);
template int convert<float, double>(long long, const float*, double*, hipStream_t);
template int convert<double, double>(long long, const double*, double*, hipStream_t);

}  // namespace ahoc
