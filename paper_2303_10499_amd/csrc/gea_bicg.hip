// gea_bicg.hip -- implicit transport of Steps 1 and 2 (Sec. 3, eqs. step2_sd
// of Step 1 and step3_sd with their convective and diffusive terms at the
// new level): the matrix-free non-symmetric operators and BiCGStab with the
// Jacobi preconditioner on the right (van der Vorst's algorithm).
//
// One operator serves both systems (times the cell volume):
//   (A x)_P = c_P x_P + gamma sum_out phi_f I4(x)_f + sum_f k_d (x_P - x_nb)
//             + sum_{wall faces along d = wall_comp} 2 k_d x_P,
// c_P = rho*_P tcoef.  Momentum component m: tcoef = V/dt, gamma = 1,
// k_d = mu S_d/h_d, wall_comp = m (the wall-normal component vanishes on the
// wall, half a spacing away).  Energy (unknown T): tcoef = c_v V/dt or
// c_p V/dt, gamma = c_p, k_d = (mu/Pr) c_p S_d/h_d, adiabatic walls.  I4 is
// the cubic face interpolation (-1, 9, 9, -1)/16 with two cells on each
// side, else the linear mean; there is no convective flux through a wall.
//
// The operator kernels march column tiles through z like the explicit step
// kernels (the line along z in registers, the x/y neighbours from the
// caches, the flux of the face below carried from the plane below); the
// vector updates are grid-stride passes.  Each kernel stores one partial a
// workgroup for every dot product it forms; every workgroup of the next
// kernel sums them in workgroup order (bitwise reproducible) and takes the
// scalars a stage on, and workgroup 0 leaves them for the kernel after it.
// (A kernel reads the scalars of one slot and writes those of another, and
// the partials of the five stages lie apart, so nothing is read while it is
// written.)  An iteration is five launches; with a one-workgroup kernel
// behind each stage it was nine, which on 100 x 100 cells, where each launch
// takes about 4.5 us whatever it does, was 40 us an iteration against 23: five
// steps with implicit transport 5.2 ms before and 3.6 now.
// All kernels of an iteration return at once when the scalars say the solve
// is done, so the host enqueues iterations in batches (the first as long as
// the last solve of that kind was) and reads the scalars once a batch.
#include <hip/hip_runtime.h>

#include "gea_internal.h"
#include "gea_reduce.h"
#include "gea_stencil.h"

namespace gea {
namespace {

template <int NDIM>
struct TrOpD {
  const double* rho_star;
  double tcoef;
  const double* phi[NDIM];
  double gamma;
  double k[NDIM];
  int wall_comp;
};

template <int NDIM>
TrOpD<NDIM> dev_op(const TrOp& o) {
  TrOpD<NDIM> d;
  d.rho_star = o.rho_star;
  d.tcoef = o.tcoef;
  d.gamma = o.gamma;
  d.wall_comp = o.wall_comp;
  for (int i = 0; i < NDIM; ++i) {
    d.phi[i] = o.phi[i];
    d.k[i] = o.k[i];
  }
  return d;
}

template <int NDIM>
Vec<NDIM> uvec(double* const* a) {
  Vec<NDIM> v;
  for (int d = 0; d < NDIM; ++d) v.p[d] = a[d];
  return v;
}

// weight of the face's lower cell (q) or upper cell in its I4 value
__device__ __forceinline__ double i4_weight(int q, int n) {
  return (q >= 1 && q + 2 <= n - 1) ? 9.0 / 16.0 : 0.5;
}

template <int N>
__device__ __forceinline__ void store_partials(double (&v)[N], double* part) {
  __shared__ double sh[N][kBlock / 64];
  Reducer<0u, N>::block(v, sh);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < N; ++k) part[k * gridDim.x + blockIdx.x] = v[k];
  }
}

// (barriers that order LDS only: the caller's loads stay in flight)
template <int N>
__device__ __forceinline__ void sum_partials(const double* part, int nb, double (&a)[N]) {
  __shared__ double sh[N][kBlock / 64];
#pragma unroll
  for (int k = 0; k < N; ++k) a[k] = 0.0;
  for (int b = threadIdx.x; b < nb; b += kBlock) {
#pragma unroll
    for (int k = 0; k < N; ++k) a[k] += part[k * nb + b];
  }
  Reducer<0u, N>::block_lds(a, sh);
}

// ---- the scalars, a stage at a time ------------------------------------------

// slots of the scalars: what the host reads, then as each kernel leaves them
enum TrSlot { kSlotHost, kSlotDir, kSlotHalf, kSlotTwo, kSlotUpdate };

// What a stage hands its kernel: whether the solve goes on, and the factor it
// formed (dir: beta, with omega beside it).
struct TrStage {
  bool go;
  double f, omega;
};

// workgroup 0 leaves the scalars `in` as f changes them
template <typename F>
__device__ __forceinline__ void leave(const TrScalars* in, TrScalars* out, F&& f) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  TrScalars sc = *in;
  f(sc);
  *out = sc;
}
__device__ __forceinline__ void tr_finish(TrScalars& sc, int status) {
  sc.status = status;
  sc.done = 1;
}

// after the set-up: ||b||^2, rho = <rh, r> = ||r||^2, the first beta
__device__ __forceinline__ TrStage tr_begin(const TrParts& q, TrScalars* slots) {
  double a[2];
  sum_partials<2>(q.setup, q.nz, a);
  const double tol2 = q.tol * q.tol;
  int status = 1;  // (goes on)
  if (!isfinite(a[0]) || !isfinite(a[1]))
    status = -5;
  else if (a[0] == 0.0 || a[1] <= tol2 * a[0])
    status = 0;  // (b = 0: the caller sets x = 0)
  else if (q.max_iter < 1 || a[1] == 0.0)
    status = -4;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    TrScalars sc;
    sc.bb = a[0];
    sc.rr = a[1];
    sc.rr0 = a[1];
    sc.rho = a[1];
    sc.rho_old = 1.0;
    sc.alpha = 1.0;
    sc.omega = 1.0;
    sc.beta = a[1];  // (rho / rho_old) (alpha / omega) with rho_old = alpha = omega = 1
    sc.tol2 = tol2;
    sc.iter = 0;
    sc.max_iter = q.max_iter;
    sc.status = status == 1 ? 0 : status;
    sc.done = status != 1;
    slots[kSlotDir] = sc;
  }
  return TrStage{status == 1, a[1], 1.0};
}

// rho_new = <rh, r>, ||r||^2: stop test, the next beta
__device__ __forceinline__ TrStage tr_end(const TrParts& q, TrScalars* slots, int to) {
  const TrScalars* const in = slots + kSlotUpdate;
  double a[2];
  sum_partials<2>(q.rhr, q.nb, a);
  const bool was = in->done;
  const double omega = in->omega, beta = (a[0] / in->rho) * (in->alpha / omega);
  int status = 1;
  if (!isfinite(a[0]) || !isfinite(a[1]))
    status = -5;
  else if (a[1] <= in->tol2 * in->bb)
    status = 0;
  else if (in->iter >= in->max_iter || omega == 0.0 || a[0] == 0.0)
    status = -4;
  leave(in, slots + to, [&](TrScalars& sc) {
    if (was) return;
    sc.rr = a[1];
    if (status != 1) {
      tr_finish(sc, status);
    } else {
      sc.beta = beta;
      sc.rho_old = sc.rho;
      sc.rho = a[0];
    }
  });
  return TrStage{!was && status == 1, beta, omega};
}

// alpha = rho / <rh, v>
__device__ __forceinline__ TrStage tr_alpha(const TrParts& q, TrScalars* slots) {
  const TrScalars* const in = slots + kSlotDir;
  double a[1];
  sum_partials<1>(q.rhv, q.nz, a);
  const bool was = in->done, bad = !(a[0] != 0.0) || !isfinite(a[0]);
  const double alpha = in->rho / a[0];
  leave(in, slots + kSlotHalf, [&](TrScalars& sc) {
    if (was) return;
    if (bad)
      tr_finish(sc, isfinite(a[0]) ? -4 : -5);
    else
      sc.alpha = alpha;
  });
  return TrStage{!was && !bad, alpha, 0.0};
}

// ||s||^2: converged after the half step?
__device__ __forceinline__ TrStage tr_half_check(const TrParts& q, TrScalars* slots) {
  const TrScalars* const in = slots + kSlotHalf;
  double a[1];
  sum_partials<1>(q.ss, q.nb, a);
  const bool was = in->done, fin = !isfinite(a[0]) || a[0] <= in->tol2 * in->bb;
  leave(in, slots + kSlotTwo, [&](TrScalars& sc) {
    if (was) return;
    sc.iter += 1;
    if (!isfinite(a[0])) {
      tr_finish(sc, -5);
    } else if (fin) {
      sc.rr = a[0];
      tr_finish(sc, 0);
    }
  });
  return TrStage{!was && !fin, 0.0, 0.0};
}

// omega = <t, s> / <t, t>
__device__ __forceinline__ TrStage tr_omega(const TrParts& q, TrScalars* slots) {
  const TrScalars* const in = slots + kSlotTwo;
  double a[2];
  sum_partials<2>(q.ts, q.nz, a);
  const bool was = in->done, bad = !(a[1] != 0.0) || !isfinite(a[0]) || !isfinite(a[1]);
  const double omega = a[0] / a[1];
  leave(in, slots + kSlotUpdate, [&](TrScalars& sc) {
    if (was) return;
    if (bad)
      tr_finish(sc, isfinite(a[1]) ? -4 : -5);
    else
      sc.omega = omega;
  });
  return TrStage{!was && !bad, omega, 0.0};
}

// The operator at cell P of a column (plane k): (A x)_P and its diagonal.
// zx holds x along the column (k-2..k+2); the x/y lines are loaded here;
// fz_lo, fz_hi are the fluxes of the faces below and above (0 on a wall).
template <int NDIM>
__device__ __forceinline__ double tr_plane(const Geo& G, const TrOpD<NDIM>& op, const Col& c,
                                           int P, int k, const double* __restrict__ x,
                                           const Line& zx, double fz_lo, double fz_hi,
                                           double* diag) {
  constexpr int Z = NDIM - 1;
  const int nz = G.n[Z];
  const double xc = zx.c;
  const double cP = op.rho_star[P] * op.tcoef;
  double conv = 0.0, cdiag = 0.0, lap = 0.0, ldiag = 0.0;
  auto faces = [&](const Line& l, int q, int n, double fh, double fl, double kd, bool wall) {
    const double wallk = wall ? 2.0 * kd : 0.0;
    if (q + 1 < n) {
      conv += fh * i4_hi(l, q, n);
      cdiag += fh * i4_weight(q, n);
      lap += kd * (xc - l.p1);
      ldiag += kd;
    } else {
      lap += wallk * xc;
      ldiag += wallk;
    }
    if (q > 0) {
      conv -= fl * i4_lo(l, q, n);
      cdiag -= fl * i4_weight(q - 1, n);
      lap += kd * (xc - l.m1);
      ldiag += kd;
    } else {
      lap += wallk * xc;
      ldiag += wallk;
    }
  };
#pragma unroll
  for (int d = 0; d < Z; ++d) {
    const int st = G.st[d], n = G.n[d], q = coord(c, d);
    const Line l = line_at([&](int Q) { return x[Q]; }, P, st, q, n);
    const double fh = op.phi[d][P], fl = op.phi[d][nb(q > 0, P - st, P)];
    faces(l, q, n, fh, fl, op.k[d], op.wall_comp == d);
  }
  faces(zx, k, nz, fz_hi, fz_lo, op.k[Z], op.wall_comp == Z);
  *diag = cP + op.gamma * cdiag + ldiag;
  return cP * xc + op.gamma * conv + lap;
}

// sum_out phi I4(w) at cell P (the explicit part of Step 2's transport)
template <int NDIM>
__device__ __forceinline__ double tr_conv(const Geo& G, const TrOpD<NDIM>& op, const Col& c, int P,
                                          int k, const double* __restrict__ w, const Line& zw,
                                          double fz_lo, double fz_hi) {
  constexpr int Z = NDIM - 1;
  double conv = 0.0;
#pragma unroll
  for (int d = 0; d < Z; ++d) {
    const int st = G.st[d], n = G.n[d], q = coord(c, d);
    const Line l = line_at([&](int Q) { return w[Q]; }, P, st, q, n);
    if (q + 1 < n) conv += op.phi[d][P] * i4_hi(l, q, n);
    if (q > 0) conv -= op.phi[d][P - st] * i4_lo(l, q, n);
  }
  const int nz = G.n[Z];
  if (k + 1 < nz) conv += fz_hi * i4_hi(zw, k, nz);
  if (k > 0) conv -= fz_lo * i4_lo(zw, k, nz);
  return conv;
}

// ---- set-up ------------------------------------------------------------------

// The set-up and operator kernels form their partials themselves (DOTS) or
// leave them to k_tr_column_dots.

// momentum component: b = V (rho^n u^n/dt - R(F^n)) from the explicit
// predictor's pass, r = b - A x0, rh = r, p = v = 0, 1/diag; partials
// ||b||^2, ||r||^2
template <int NDIM, bool DOTS>
__global__ __launch_bounds__(kBlock) void k_tr_setup_mom(Geo G, int kc, TrOpD<NDIM> op,
                                                         const double* __restrict__ x0, TrVecs v,
                                                         double* part) {
  constexpr int Z = NDIM - 1;
  const Col c = col_of<NDIM>(G, kc);
  double red[2] = {0.0, 0.0};
  if (c.act) {
    const int nz = G.n[Z], pl = c.pl;
    int P = c.base + pl * c.k0;
    Line zx = line_at([&](int Q) { return x0[Q]; }, P, pl, c.k0, nz);
    double flo = c.k0 > 0 ? op.phi[Z][P - pl] : 0.0;
    for (int k = c.k0; k < c.k1; ++k, P += pl) {
      const double fhi = op.phi[Z][P];
      const double xn = x0[nb(k + 3 < nz, P + 3 * pl, P)];
      double diag;
      const double ax = tr_plane<NDIM>(G, op, c, P, k, x0, zx, flo, fhi, &diag);
      const double b = v.b[P], r = b - ax;
      v.dinv[P] = 1.0 / diag;
      v.r[P] = r;
      v.rh[P] = r;
      v.p[P] = 0.0;
      v.v[P] = 0.0;
      if (DOTS) {
        red[0] += b * b;
        red[1] += r * r;
      }
      flo = fhi;
      zx = shift(zx, k + 3 < nz ? xn : 0.0);
    }
  }
  if constexpr (DOTS) store_partials<2>(red, part);
}

// the known part of Step 2's transported quantity: K* (+ Phi in the
// total-energy form)
template <int NDIM>
__global__ __launch_bounds__(kBlock) void k_tr_known(Geo G, Phys ph, Vec<NDIM> u_star, int enth,
                                                     double* __restrict__ w) {
  GEA_FOR_CELLS(P, G) {
    double kin = 0.0;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) kin += u_star.p[d][P] * u_star.p[d][P];
    const int kz = P / G.st[NDIM - 1];
    w[P] = 0.5 * kin + (enth ? 0.0 : ph.g * (kz + 0.5) * G.dz);
  }
}

// energy: b = local - sum_out phi I4(w) + bg, local = V/dt (rho^n e^n - rho* w)
// (total energy, e0 = e^n) or V/dt q (enthalpy form, e0 = q); x = T^n (the
// initial guess, written into the solution buffer), r = b - A x, rh = r,
// p = v = 0; partials ||b||^2, ||r||^2
template <int NDIM, bool ENTH, bool DOTS>
__global__ __launch_bounds__(kBlock) void k_tr_setup_energy(
    Geo G, Phys ph, int kc, TrOpD<NDIM> op, const double* __restrict__ rho,
    const double* __restrict__ e0, const double* __restrict__ w, const double* __restrict__ Tn,
    const double* __restrict__ Tbg, double* __restrict__ x, TrVecs v, double* part) {
  constexpr int Z = NDIM - 1;
  const Col c = col_of<NDIM>(G, kc);
  double red[2] = {0.0, 0.0};
  if (c.act) {
    const int nz = G.n[Z], pl = c.pl;
    const double kdz = op.k[Z];   // (mu/Pr) c_p S_z/h_z
    int P = c.base + pl * c.k0;
    Line zT = line_at([&](int Q) { return Tn[Q]; }, P, pl, c.k0, nz);
    Line zw = line_at([&](int Q) { return w[Q]; }, P, pl, c.k0, nz);
    double flo = c.k0 > 0 ? op.phi[Z][P - pl] : 0.0;
    for (int k = c.k0; k < c.k1; ++k, P += pl) {
      const double fhi = op.phi[Z][P];
      const int Pn = nb(k + 3 < nz, P + 3 * pl, P);
      const double Tnext = Tn[Pn], wnext = w[Pn];
      const double rs = op.rho_star[P];
      const double local = ENTH ? G.V / ph.dt * e0[P] : G.V / ph.dt * (rho[P] * e0[P] - rs * zw.c);
      const double convw = tr_conv<NDIM>(G, op, c, P, k, w, zw, flo, fhi);
      double bg = 0.0;
      if (k + 1 < nz) bg += kdz * (Tbg[k] - Tbg[k + 1]);
      if (k > 0) bg += kdz * (Tbg[k] - Tbg[k - 1]);
      const double b = local - convw + bg;
      double diag;
      const double ax = tr_plane<NDIM>(G, op, c, P, k, Tn, zT, flo, fhi, &diag);
      const double r = b - ax;
      x[P] = zT.c;
      v.b[P] = b;
      v.dinv[P] = 1.0 / diag;
      v.r[P] = r;
      v.rh[P] = r;
      v.p[P] = 0.0;
      v.v[P] = 0.0;
      if (DOTS) {
        red[0] += b * b;
        red[1] += r * r;
      }
      flo = fhi;
      const bool more = k + 3 < nz;
      zT = shift(zT, more ? Tnext : 0.0);
      zw = shift(zw, more ? wnext : 0.0);
    }
  }
  if constexpr (DOTS) store_partials<2>(red, part);
}

// ---- one iteration -----------------------------------------------------------

// (The vector passes load their first cell before the scalars' sums, whose
// latency is as long: on 150 x 90 x 61 cells k_tr_half takes 10 us, as it did
// with the sums in a launch of 5 us before it, and 21 without.)

// p = r + beta (p - omega v), y = dinv p.  FROM: where the scalars come from:
// 0 the host's slot (a batch goes on), 1 the update before, 2 the set-up
template <int FROM>
__global__ __launch_bounds__(kBlock) void k_tr_dir(int nc, TrVecs v, TrParts q, TrScalars* slots) {
  int P = blockIdx.x * blockDim.x + threadIdx.x;
  const int P0 = P < nc ? P : nc - 1;
  double r = v.r[P0], p = v.p[P0], vv = v.v[P0], di = v.dinv[P0];
  TrStage st;
  if constexpr (FROM == 0) {
    const TrScalars* const in = slots + kSlotHost;
    st = TrStage{in->done == 0, in->beta, in->omega};
    leave(in, slots + kSlotDir, [](TrScalars&) {});
  } else {
    st = FROM == 1 ? tr_end(q, slots, kSlotDir) : tr_begin(q, slots);
  }
  if (!st.go) return;
  for (; P < nc;) {
    const double pn = r + st.f * (p - st.omega * vv);
    v.p[P] = pn;
    v.y[P] = di * pn;
    P += gridDim.x * blockDim.x;
    if (P >= nc) break;
    r = v.r[P], p = v.p[P], vv = v.v[P], di = v.dinv[P];
  }
}

// out = A in (TWO = 0: v = A y, partial <rh, v>; TWO = 1: t = A z, partials
// <t, s>, <t, t> with s in r)
template <int NDIM, int TWO, bool DOTS>
__global__ __launch_bounds__(kBlock) void k_tr_matvec(Geo G, int kc, TrOpD<NDIM> op,
                                                      const double* __restrict__ in,
                                                      double* __restrict__ out,
                                                      const double* __restrict__ dv, TrParts q,
                                                      TrScalars* slots) {
  if (TWO) {
    if (!tr_half_check(q, slots).go) return;
  } else {
    if (slots[kSlotDir].done) return;
  }
  constexpr int Z = NDIM - 1;
  const Col c = col_of<NDIM>(G, kc);
  double red[2] = {0.0, 0.0};
  if (c.act) {
    const int nz = G.n[Z], pl = c.pl;
    int P = c.base + pl * c.k0;
    Line zx = line_at([&](int Q) { return in[Q]; }, P, pl, c.k0, nz);
    double flo = c.k0 > 0 ? op.phi[Z][P - pl] : 0.0;
    for (int k = c.k0; k < c.k1; ++k, P += pl) {
      const double fhi = op.phi[Z][P];
      const double xn = in[nb(k + 3 < nz, P + 3 * pl, P)];
      const double d = DOTS ? dv[P] : 0.0;
      double diag;
      const double a = tr_plane<NDIM>(G, op, c, P, k, in, zx, flo, fhi, &diag);
      out[P] = a;
      if (!DOTS) {
      } else if (TWO) {
        red[0] += a * d;
        red[1] += a * a;
      } else {
        red[0] += d * a;
      }
      flo = fhi;
      zx = shift(zx, k + 3 < nz ? xn : 0.0);
    }
  }
  if (!DOTS) return;
  if (TWO) {
    store_partials<2>(red, q.ts);
  } else {
    double one[1] = {red[0]};
    store_partials<1>(one, q.rhv);
  }
}

// The partials of those kernels in the order of the fixed chunks (kc planes a
// thread), from the stored vectors: KIND 0 <b, a>; 1 <a, b>, <a, a>; 2 <a, a>,
// <b, b>.  slot: returns at once when its scalars say done (-1: never).
template <int KIND>
__global__ __launch_bounds__(kBlock) void k_tr_column_dots(Geo G, int kc, const double* __restrict__ a,
                                                           const double* __restrict__ b,
                                                           const TrScalars* slots, int slot, double* part) {
  if (slot >= 0 && slots[slot].done) return;
  const Col c = col_of<3>(G, kc);
  double red[2] = {0.0, 0.0};
  if (c.act) {
    const double* pa = a + c.base + (long)c.pl * c.k0;
    const double* pb = b + c.base + (long)c.pl * c.k0;
    auto add = [&](double x, double y) {
      if (KIND == 0) {
        red[0] += y * x;
      } else if (KIND == 1) {
        red[0] += x * y;
        red[1] += x * x;
      } else {
        red[0] += x * x;
        red[1] += y * y;
      }
    };
    constexpr int U = 16;  // planes in flight
    int k = c.k0;
    for (; k + U <= c.k1; k += U) {
      double x[U], y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        x[u] = *pa;
        y[u] = *pb;
        pa += c.pl;
        pb += c.pl;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add(x[u], y[u]);
    }
    for (; k < c.k1; ++k, pa += c.pl, pb += c.pl) add(*pa, *pb);
  }
  if constexpr (KIND == 0) {
    double one[1] = {red[0]};
    store_partials<1>(one, part);
  } else {
    store_partials<2>(red, part);
  }
}

// x += alpha y, s = r - alpha v (into r), z = dinv s; partial ||s||^2
__global__ __launch_bounds__(kBlock) void k_tr_half(int nc, double* __restrict__ x, TrVecs v,
                                                    TrParts q, TrScalars* slots) {
  int P = blockIdx.x * blockDim.x + threadIdx.x;
  const int P0 = P < nc ? P : nc - 1;
  double xv = x[P0], y = v.y[P0], r = v.r[P0], vv = v.v[P0], di = v.dinv[P0];
  const TrStage st = tr_alpha(q, slots);
  if (!st.go) return;
  const double alpha = st.f;
  double red[1] = {0.0};
  for (; P < nc;) {
    x[P] = xv + alpha * y;
    const double s = r - alpha * vv;
    v.r[P] = s;
    v.z[P] = di * s;
    red[0] += s * s;
    P += gridDim.x * blockDim.x;
    if (P >= nc) break;
    xv = x[P], y = v.y[P], r = v.r[P], vv = v.v[P], di = v.dinv[P];
  }
  store_partials<1>(red, q.ss);
}

// x += omega z, r = s - omega t; partials <rh, r>, ||r||^2
__global__ __launch_bounds__(kBlock) void k_tr_update(int nc, double* __restrict__ x, TrVecs v,
                                                      TrParts q, TrScalars* slots) {
  int P = blockIdx.x * blockDim.x + threadIdx.x;
  const int P0 = P < nc ? P : nc - 1;
  double xv = x[P0], z = v.z[P0], s = v.r[P0], t = v.t[P0], rh = v.rh[P0];
  const TrStage st = tr_omega(q, slots);
  if (!st.go) return;
  const double omega = st.f;
  double red[2] = {0.0, 0.0};
  for (; P < nc;) {
    x[P] = xv + omega * z;
    const double r = s - omega * t;
    v.r[P] = r;
    red[0] += rh * r;
    red[1] += r * r;
    P += gridDim.x * blockDim.x;
    if (P >= nc) break;
    xv = x[P], z = v.z[P], s = v.r[P], t = v.t[P], rh = v.rh[P];
  }
  store_partials<2>(red, q.rhr);
}

// the scalars behind the last kernel of a batch, for the host
__global__ __launch_bounds__(kBlock) void k_tr_end(TrParts q, TrScalars* slots) {
  tr_end(q, slots, kSlotHost);
}

}  // namespace

// ---- launchers ---------------------------------------------------------------

static ZPlan tr_plan(const Geo& G, const TrOp& op) { return op.fixed_order ? zplan_fixed(G) : zplan(G); }

// Chunks of the fixed order leave CUs idle on 3D meshes of few columns, where
// a thread's chain of 64 planes is all latency.  There the operator kernels
// take the chunks that fill the card, and their sums a pass of their own in
// the fixed order: on 150 x 90 x 61 cells (69 workgroups) k_tr_matvec
// went from 45 to 18 + 8 us, the set-up of a momentum component from 55 to
// 23 + 8 and of the energy solve from 97 to 37 + 8.  (Four threads a column in
// one workgroup, the first summing what all had stored: 24-32 us.)
static bool dots_apart(const Geo& G, const TrOp& op) {
  return G.ndim == 3 && op.fixed_order && zplan(G).kc < zplan_fixed(G).kc;
}

namespace {

// the partials of the stages, apart from each other in one area
TrParts tr_parts(const Geo& G, const TrOp& op, double* part, double tol, int max_iter) {
  TrParts q;
  q.nb = grid_for(G.nc);
  q.nz = tr_plan(G, op).blocks;
  q.rhv = part;
  q.ts = q.rhv + q.nz;
  q.ss = q.ts + 2L * q.nz;
  q.rhr = q.ss + q.nb;
  q.setup = q.rhr + 2L * q.nb;
  q.tol = tol;
  q.max_iter = max_iter;
  return q;
}

}  // namespace

long tr_part_doubles(const Geo& G) {
  const int a = zplan(G).blocks, b = zplan_fixed(G).blocks;
  return 5L * (a > b ? a : b) + 3L * grid_for(G.nc);
}

namespace {

template <int KIND>
void column_dots(hipStream_t s, const Geo& G, const double* a, const double* b, const TrScalars* slots,
                 int slot, double* part) {
  const ZPlan zf = zplan_fixed(G);
  hipLaunchKernelGGL(k_tr_column_dots<KIND>, dim3(zf.blocks), dim3(kBlock), 0, s, G, zf.kc, a, b, slots, slot, part);
}

template <int NDIM>
void setup_mom(hipStream_t s, const Geo& G, const TrOp& op, const double* x0, const TrVecs& v, double* to) {
  if constexpr (NDIM == 3)
    if (dots_apart(G, op)) {
      const ZPlan zp = zplan(G);
      hipLaunchKernelGGL((k_tr_setup_mom<3, false>), dim3(zp.blocks), dim3(kBlock), 0, s, G, zp.kc, dev_op<3>(op), x0, v, to);
      column_dots<2>(s, G, v.b, v.r, nullptr, -1, to);
      return;
    }
  const ZPlan zp = tr_plan(G, op);
  hipLaunchKernelGGL((k_tr_setup_mom<NDIM, true>), dim3(zp.blocks), dim3(kBlock), 0, s, G, zp.kc, dev_op<NDIM>(op), x0, v, to);
}

template <int NDIM, bool ENTH>
void setup_energy(hipStream_t s, const Geo& G, const Phys& ph, const TrOp& op, const double* rho,
                  const double* e0, const double* w, const double* Tn, const double* Tbg, double* x,
                  const TrVecs& v, double* to) {
  if constexpr (NDIM == 3)
    if (dots_apart(G, op)) {
      const ZPlan zp = zplan(G);
      hipLaunchKernelGGL((k_tr_setup_energy<3, ENTH, false>), dim3(zp.blocks), dim3(kBlock), 0, s, G, ph, zp.kc, dev_op<3>(op), rho, e0, w, Tn, Tbg, x, v, to);
      column_dots<2>(s, G, v.b, v.r, nullptr, -1, to);
      return;
    }
  const ZPlan zp = tr_plan(G, op);
  hipLaunchKernelGGL((k_tr_setup_energy<NDIM, ENTH, true>), dim3(zp.blocks), dim3(kBlock), 0, s, G, ph, zp.kc, dev_op<NDIM>(op), rho, e0, w, Tn, Tbg, x, v, to);
}

template <int NDIM, int TWO>
void matvec(hipStream_t s, const Geo& G, const TrOp& op, const double* in, double* out,
            const double* dv, const TrParts& q, TrScalars* slots) {
  if constexpr (NDIM == 3)
    if (dots_apart(G, op)) {
      const ZPlan zp = zplan(G);
      hipLaunchKernelGGL((k_tr_matvec<3, TWO, false>), dim3(zp.blocks), dim3(kBlock), 0, s, G, zp.kc, dev_op<3>(op), in, out, dv, q, slots);
      column_dots<TWO>(s, G, out, dv, slots, TWO ? kSlotTwo : kSlotDir, TWO ? q.ts : q.rhv);
      return;
    }
  const ZPlan zp = tr_plan(G, op);
  hipLaunchKernelGGL((k_tr_matvec<NDIM, TWO, true>), dim3(zp.blocks), dim3(kBlock), 0, s, G, zp.kc, dev_op<NDIM>(op), in, out, dv, q, slots);
}

}  // namespace

void launch_tr_setup_mom(hipStream_t s, const Geo& G, const TrOp& op, const double* x0,
                         const TrVecs& v, double* part) {
  (G.ndim == 2 ? setup_mom<2> : setup_mom<3>)(s, G, op, x0, v, tr_parts(G, op, part, 0.0, 0).setup);
}

void launch_tr_setup_energy(hipStream_t s, const Geo& G, const Phys& ph, bool enth, const TrOp& op,
                            const double* rho, const double* e0, double* const* u_star,
                            double* w, const double* Tn, const double* Tbg, double* x,
                            const TrVecs& v, double* part) {
  const int gb = grid_for(G.nc);
  double* const to = tr_parts(G, op, part, 0.0, 0).setup;
  if (G.ndim == 2) {
    hipLaunchKernelGGL(k_tr_known<2>, dim3(gb), dim3(kBlock), 0, s, G, ph, uvec<2>(u_star), (int)enth, w);
    (enth ? setup_energy<2, true> : setup_energy<2, false>)(s, G, ph, op, rho, e0, w, Tn, Tbg, x, v, to);
  } else {
    hipLaunchKernelGGL(k_tr_known<3>, dim3(gb), dim3(kBlock), 0, s, G, ph, uvec<3>(u_star), (int)enth, w);
    (enth ? setup_energy<3, true> : setup_energy<3, false>)(s, G, ph, op, rho, e0, w, Tn, Tbg, x, v, to);
  }
}

void launch_tr_iterations(hipStream_t s, const Geo& G, const TrOp& op, double* x, const TrVecs& v,
                          double* part, TrScalars* slots, double tol, int max_iter, int n, bool first) {
  const TrParts q = tr_parts(G, op, part, tol, max_iter);
  const dim3 grid(q.nb), block(kBlock);
  const auto mv0 = G.ndim == 2 ? matvec<2, 0> : matvec<3, 0>, mv1 = G.ndim == 2 ? matvec<2, 1> : matvec<3, 1>;
  for (int k = 0; k < n; ++k) {
    if (k > 0)
      hipLaunchKernelGGL(k_tr_dir<1>, grid, block, 0, s, G.nc, v, q, slots);
    else if (first)
      hipLaunchKernelGGL(k_tr_dir<2>, grid, block, 0, s, G.nc, v, q, slots);
    else
      hipLaunchKernelGGL(k_tr_dir<0>, grid, block, 0, s, G.nc, v, q, slots);
    mv0(s, G, op, v.y, v.v, v.rh, q, slots);
    hipLaunchKernelGGL(k_tr_half, grid, block, 0, s, G.nc, x, v, q, slots);
    mv1(s, G, op, v.z, v.t, v.r, q, slots);
    hipLaunchKernelGGL(k_tr_update, grid, block, 0, s, G.nc, x, v, q, slots);
  }
  hipLaunchKernelGGL(k_tr_end, dim3(1), block, 0, s, q, slots);
}

}  // namespace gea
