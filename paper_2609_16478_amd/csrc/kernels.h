// Host-side launchers of the stencil, setup and Krylov kernels.
#pragma once

#include "common.h"

namespace ahoc {

// stencil.hip -------------------------------------------------------------------------
template <typename T>
int lift(const Geom& g, const Weights& w, const T* Q, const T* src, T* G, hipStream_t st);
template <typename T>
int rhs_u(const Geom& g, const Weights& w, const T* V, const T* Q, const T* ia, const T* src, T* G,
          hipStream_t st);
template <typename T>
int gather(const Geom& g, const Weights& w, const T* U, const T* Q, const T* af, const T* srcq,
           double* R, hipStream_t st);
// face layers of the homogeneous lift (input of the spectral lift); fixed-order sums of partials
template <typename T>
int face_lift(const Geom& g, const Weights& w, const T* Q, T* Lx, T* Ly, T* Lz, hipStream_t st);
// 3-D: the V-solve's lift layers (weights wv, layouts of face_lift) and the layers mq Q_b of the
// U-solve's source (spectral M; mq = m1 / alpha_b in Q layout), layouts as face_lift except the y
// faces, [2][n_x'][n_z'] (z fastest), in one tiled pass over Q
template <typename T> struct FaceLiftW {
  T w0[3], wf[3], ws[3];  // per face axis: normal, faster and slower tangential couplings
};
template <typename T>
int face_lifts3(const Geom& g, const Weights& wv, const T* Q, const T* mq, T* Lx, T* Ly, T* Lz, T* Ux, T* Uy,
                T* Uz, hipStream_t st);
// 2-D: the same two sets (layouts of face_lift; ia nodal 1/alpha) in one pass over Q
template <typename T>
int face_lifts2(const Geom& g, const Weights& wv, const T* Q, const T* ia, T* Lx, T* Ly, T* Ux, T* Uy, hipStream_t st);
// out[q] = s * nodal(boundary node of q): a nodal field in Q layout
template <typename T>
int nodal_to_q(const Geom& g, double s, const T* nodal, T* out, hipStream_t st);
template <typename T>
int partial_sum(long long n, int count, long long stride, const T* in, T* out, hipStream_t st);
// boundary-symbol preconditioner (precond.hip): inverse 2x2 block coefficients per face
// mode from per-axis FP64 tables {s, cos, sin, w_lo} x 3 axes, and their application to
// face spectra of a Q-layout vector
// (tri: the triharmonic chain and q-row; tabs then hold its fourth-derivative combination
// a_1 sin(pi k/N) + ... + a_4 sin(4 pi k/N) in place of w_lo)
int precond_symbol(const Geom& g, const Weights& w, double c, int navier, const double* const* tabs, double* pc,
                   double* qc, hipStream_t st, bool tri = false);
template <typename T>
int precond_modes(const Geom& g, const T* pc, const T* qc, T* x, hipStream_t st);
// boundary residual from face sums formed in spectral space
template <typename T>
int gather_faces(const Geom& g, const T* Fx, const T* Fy, const T* Fz, const T* Q, const T* af,
                 const T* srcq, double* R, hipStream_t st);
template <typename T>
int resid64(const Geom& g, const Weights& w, const double* U, const double* V, const double* Q,
            const double* ia, const double* af, const double* src_u, const double* src_v,
            const double* src_q, T* ru, T* rv, T* rq, hipStream_t st);
int setup_inv_alpha(long long n, const double* alpha, double* ia64, float* ia32, double* bmin,
                    int nb, hipStream_t st);
int setup_face_alpha(const Geom& g, const double* alpha, double* af64, float* af32, hipStream_t st);
// variable shift c (nodal): y = -L_h[V] + M(c V) on the interior of a single problem, V = X there
// and zero on the boundary: 2-D, and 3-D with the work-groups' parts of <u, y> in part[0..nb) and
// of <y, y> in part[nb..2 nb), nb = vapply_dot_blocks (0 in 2-D; y's row padding is left as it is)
int vapply(const Geom& g, const Weights& w, const double* X, const double* c, double* y, hipStream_t st);
int vapply_dot_blocks(const Geom& g);
int vapply_dot(const Geom& g, const Weights& w, const double* X, const double* c, double* y, const double* u,
               double* part, hipStream_t st);
// the V-solve's start on n = the padded interior: r = rh = p = src - A V with V = Q on the face
// interiors and 0 inside (src may be null), and nb parts of <r, r>
int vstart(const Geom& g, const Weights& w, long long n, const double* Q, const double* c, const double* src, double* r,
           double* rh, double* p, double* part, int nb, hipStream_t st);
// per-block min and max (part[2 b], part[2 b + 1]) of n doubles
int minmax_partial(long long n, const double* x, double* part, int nblocks, hipStream_t st);
// Navier faces (the same on every instance of a batch): af = 0 and src_q = -alpha g_L on
// their q-rows
int setup_navier(const Geom& g, int mask, const double* alpha, const double* gL, double* af64, float* af32,
                 double* src_q, hipStream_t st);
// triharmonic extension: interior sources of the W-, V- and U-solves, the q-rows' known part
// and face coefficient, and the boundary residual R = af h^-4 sum a_k U_k - Q - src_q
int tri_sources(const Geom& g, const Weights& w, const double* f, const double* gD, const double* lapu,
                const double* bilap, double* sw, double* sv, double* su, hipStream_t st);
int tri_srcq(const Geom& g, int mask, const double* gD, const double* gN, const double* gNN, const double* tang4,
             const double* bilap, double* src_q, double* af64, float* af32, hipStream_t st);
template <typename T>
int gather_tri(const Geom& g, const T* U, const T* Q, const T* af, const T* srcq, double* R, hipStream_t st);
int setup_sources(const Geom& g, const Weights& w, const double* f, const double* alpha,
                  const double* gD, const double* gN, const double* lapgD, double* src_v,
                  double* src_u, double* src_q, hipStream_t st);
template <typename T>
int out_u(const Geom& g, const T* Ui, const double* gD, double* u, hipStream_t st);
template <typename T>
int out_v(const Geom& g, const T* Vi, const double* Q, const double* vedge, double* v, hipStream_t st);
int mul(long long n, const double* a, const double* b, double* out, hipStream_t st);
template <typename Ti, typename To>
int pitch_copy(long long rows, int cols, const Ti* in, long long ip, To* out, long long op, hipStream_t st, int wide = 0);
template <typename Ti, typename To> int convert(long long n, const Ti* in, To* out, hipStream_t st);
template <typename Tx> int accumulate(long long n, const Tx* x, double* y, hipStream_t st);
template <typename Tx>
int absmax_partial(long long n, const Tx* x, double* bmax, int nb, hipStream_t st);
int fill(long long n, double v, double* x, hipStream_t st);

// faces2d.hip ----------------------------------------------------------------------------
// The boundary lines of a 2-D operator application on a square grid of one of the specialised
// lengths up to 1024 (lines2d_supported), one work-group per instance: everything before the
// V-solve's spectrum is generated, and everything after the face sums (see the file).
template <typename T> struct Front2d {
  const double* q;        // nb x 4 (N-1)
  double* z;              // P^-1 q, or null
  T* zt;                  // the same in T, or null
  const double *pc, *qc;  // mode blocks (Q layout), null without the preconditioner
  const cx<double>* twd;
  const double* snd;
  const cx<T>* tw;
  const T* sn;
  const T* ia;            // nodal 1/alpha
  long long nnodal;
  T w0x, w0y, wt, m1;
  T *Fx, *Fy, *Ux, *Uy;
  int px;
};
template <typename T> struct Back2d {
  const T *Fx, *Fy, *z, *af;
  const cx<T>* tw;
  const T* sn;
  double* R;
  T ihx2, ihy2;
  int px;
};
bool lines2d_supported(int N);
template <typename T> int front2d(int N, const Front2d<T>& a, int nb, hipStream_t st);
template <typename T> int back2d(int N, const Back2d<T>& a, int nb, hipStream_t st);

// poisson_small.hip ---------------------------------------------------------------------
// w = L_int^{-1} g on the dense interior of a small 2-D grid (poisson_small_ok), one launch;
// w may equal g.  sn, s: an axis's sine table (half: j <= N/2) and eigenvalues, or null, then
// they are evaluated in FP64 from n and h.
template <typename T> struct PoissonSmall {
  const double* g;
  double* w;
  int n[2];
  double h[2];
  const T* sn[2];
  const T* s[2];
  int half[2];
  T c_ta, scale;
};
template <typename T> bool poisson_small_ok(int n0, int n1);
template <typename T> int poisson_small(const PoissonSmall<T>& a, hipStream_t st);

// krylov.hip --------------------------------------------------------------------------
// partial dot products of nvec basis vectors (row stride ld) with w: part[v * nb + b]
int mdot_partial(const double* V, long long ld, int nvec, const double* w, long long n, int ns, double* part,
                 int nbk, hipStream_t st);
int mdot_reduce(const double* part, int nbk, int nvec, int ns, double* out, int ostride, int accumulate,
                hipStream_t st);
// out[s * ostride + v] = <V_v, w> over segment s: partial sums over nbk blocks and their
// reduction, or with nbk == 1 the one block's sums written directly
int mdot(const double* V, long long ld, int nvec, const double* w, long long n, int ns, double* part, int nbk,
         double* out, int ostride, hipStream_t st);
int maxpy(double* w, const double* V, long long ld, int nvec, const double* coef, int cstride, double sign,
          long long n, int ns, hipStream_t st);
int axpby(long long n, double a, const double* x, double b, double* y, hipStream_t st);
// BiCGSTAB's vector steps with their scalars kept on the device.  part holds the nb1 work-groups'
// parts of the dot products before the step (one vector after the other), part2 receives nb2
// parts of those after it; coef = {alpha, alpha is good, omega, omega is good}.
//   half:  alpha = rho / <rh, v>, r -= alpha v; <r, r>.  Neither r nor coef[0] is good where the
//          divisor is zero or not finite.
//   full:  omega = <r, t> / <t, t>, x += alpha y + omega z, r -= omega t; <rh, r>, <r, r>.  Where
//          omega is not good, x += alpha y alone.
//   to_host: the nvec sums of part and coef into the pinned out[0..nvec), out[4..8).
int bicg_half(long long n, double rho, const double* part, int nb1, const double* v, double* r, double* coef,
              double* part2, int nb2, hipStream_t st);
int bicg_full(long long n, const double* part, int nb1, const double* y, const double* z, const double* t,
              const double* rh, double* x, double* r, double* coef, double* part2, int nb2, hipStream_t st);
int bicg_to_host(const double* part, int nb, int nvec, const double* coef, double* out, hipStream_t st);
// w = a x + b y + c w
int lin3(long long n, double a, const double* x, double b, const double* y, double c, double* w, hipStream_t st);
// Segment-wise batch utilities (grid.y = segment): x_s = 0 where keep[s] == 0; gather of
// per-instance arrays (device table of device pointers, null = zeros); scatter to them.
int zero_masked(double* x, long long n, int ns, const int* keep, hipStream_t st);
int gather_ptrs(const double* const* src, long long n, int ns, double* out, hipStream_t st);
int scatter_ptrs(const double* in, long long n, int ns, double* const* dst, hipStream_t st);
int back_solve(int ns, const double* H, int m, const double* gv, const int* kk, int kmax, double* y,
               hipStream_t st);
// Arnoldi step j of ns segments of length n, ld apart in the basis V: classical Gram-Schmidt
// twice, the Givens rotation with the device-side convergence bookkeeping (see rotate_and_update in
// krylov.hip; ist = [act | kk | nit | flag | hcnt], ns ints each; hist: 16 doubles per
// instance; eres: last active estimate) and the scaling of V_{j+1}, which holds the operator's
// output on entry.  part: 2 ns (m + 1) arnoldi_slices(n) doubles; act0: ns ints of scratch.
struct ArnoldiArgs {
  int ns, m, j, max_iters;
  bool inexact;
  double tol;
  double *H, *cs, *sn, *gv, *resid;
  const double* bnorm;
  int *ist, *act0;
  double *hist, *eres, *h1, *h2, *nrm, *part;
};
// A segment up to here is one work-group's step.  A whole operator application and step in FP64,
// one work-group against slices, cycles of 12 and of 30 vectors: 380 unknowns 111 and 122, 102 and
// 119 us; 1020 97 and 112, 88 and 107; 2044 112 and 127, 106 and 122.  Beyond, the registers hold 8
// basis vectors and one compute unit reads the others from L2 four times: 3068 174 and 175, 183 and
// 166; 4092 170 and 172, 187 and 167.
constexpr long long ARN_ONE_MAX = 2048;
constexpr int ARN_INLINE = 256;          // most partial sums that every work-group adds up itself
int arnoldi_slices(long long n);
int arnoldi_step(double* V, long long ld, long long n, const ArnoldiArgs& a, hipStream_t st);
int fill_int(int* p, long long n, int v, hipStream_t st);
int start_cycle(double* v0, const double* r, long long n, int ns, const double* nrm2, double* gv, int m,
                double* beta, hipStream_t st);

}  // namespace ahoc
