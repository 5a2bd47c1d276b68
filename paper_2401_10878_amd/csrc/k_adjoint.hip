// Discrete adjoint (reverse mode) of the coupled time step, FP64, fully
// periodic boxes.
//
// Forward step t, as the step kernels compute it (Sec. 4.4, Algorithm 1):
//   f_t      = stream(f*_{t-1})                           eq. (11)
//   F_h, T_h = momentum exchange over the nodes owned by each particle in
//              o_{t-1}, with f*_{t-1}, f_t and u_p at P_{t-1}   eqs. (16)-(18)
//   P_t      = move(P_{t-1}, F_h + F_c, s)                 eqs. (2)-(3)
//   o_t      = owner map at P_t                            (Sec. 3.2)
//   f*_t     = collide(f_t, B(d_{o_t}), u_p(P_t), a(s))    eqs. (10)-(15)
// The adjoint runs these in reverse with the owner maps o and the contact
// forces F_c, T_c of the recorded forward run held fixed (the discrete
// decisions of the forward pass are not differentiated).  Orientation
// adjoints are world-frame rotation vectors: a perturbation of R is
// exp([dtheta]x) R.
//
// The reverse of a step t (from dJ/df_t and the particle adjoints Pbar_t) is
// three kernels:
//   k_adj_move     per particle: Pbar_t -> Pbar_{t-1}, dJ/dF_h, dJ/dT_h, dJ/ds
//   k_adj_mea      per node owned in o_{t-1}: the post-stream terms of the
//                  momentum exchange into dJ/df_t, and its u_p and r terms
//                  into Pbar_{t-1}
//   k_adj_collide  per node: dJ/df*_{t-1} at x, pulled from dJ/df_t at x + c_i
//                  (streaming in reverse) plus the own terms of the momentum
//                  exchange; then the collision t-1 in reverse: dJ/df_{t-1},
//                  and the coupling terms (B, u_p) into Pbar_{t-1} and into
//                  the adjoint of the fluid acceleration
#include "context.h"

// No integer decision is taken from a floating-point value in this file.
#pragma clang fp contract(fast)

namespace hlbm {

namespace {

// Particle adjoint slots: X (0-2), theta (3-5), U (6-8), omega (9-11).
constexpr int PB = 12;

// Wavefront aggregation of per-lane particle adjoint increments v[PB] keyed
// by particle id q (-1 = none): per distinct id two reduce-scatters of six
// sums (each lands in one even lane) and one FP64 atomic per sum.
__device__ void commit_adjoint(int q, const double* v, double* dst) {
  const int lane = threadIdx.x % WAVE;
  bool pend = q >= 0;
  for (;;) {
    const uint64_t m = __ballot(pend);
    if (m == 0) break;
    const int pick = __builtin_amdgcn_readlane(q, __ffsll((long long)m) - 1);
    const bool take = pend && q == pick;
    double t[PB];
    for (int k = 0; k < PB; ++k) t[k] = take ? v[k] : 0.0;
    const double s0 = wave_sum6_scatter(t), s1 = wave_sum6_scatter(t + 6);
    if (lane < 12 && (lane & 1) == 0) {
      atomic_add_f64(&dst[PB * pick + (lane >> 1)], s0);
      atomic_add_f64(&dst[PB * pick + 6 + (lane >> 1)], s1);
    }
    if (take) pend = false;
  }
}

// Record layout of one particle state: X 3, q 4, U 3, W 3, R 9.
constexpr int PREC_N = 22;
__device__ inline const double* rec_X(const double* r) { return r; }
__device__ inline const double* rec_U(const double* r) { return r + 7; }
__device__ inline const double* rec_W(const double* r) { return r + 10; }
__device__ inline const double* rec_R(const double* r) { return r + 13; }

__device__ inline void cross(const double* a, const double* b, double* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ inline void lever(const Geom& g, int x, int y, int z, const double* X, double* r) {
  r[0] = minimg((double)x - X[0], (double)g.nx, true);
  r[1] = minimg((double)y - X[1], (double)g.ny, true);
  r[2] = minimg((double)z - X[2], (double)g.nz, true);
}

// Adjoint of the momentum exchange on particle q seen from a node: r, u_p and
// Sbar = -(Fbar + Tbar x r), with Fbar, Tbar the adjoints of F_h, T_h.
struct Exchange {
  double r[3], up[3], W[3], T[3], Sb[3];
};
__device__ inline Exchange exchange_at(const Geom& g, int q, int x, int y, int z,
                                       const double* prec, const double* fhbar) {
  Exchange e;
  const double* pr = prec + (size_t)PREC_N * q;
  const double* Fb = fhbar + 6 * q;
  lever(g, x, y, z, rec_X(pr), e.r);
  for (int k = 0; k < 3; ++k) {
    e.W[k] = rec_W(pr)[k];
    e.T[k] = Fb[3 + k];
  }
  double wr[3], tr[3];
  cross(e.W, e.r, wr);
  cross(e.T, e.r, tr);
  for (int k = 0; k < 3; ++k) {
    e.up[k] = rec_U(pr)[k] + wr[k];
    e.Sb[k] = -(Fb[k] + tr[k]);
  }
  return e;
}
// c_i . (a, b, c) from the non-zero components of c_i only
__device__ inline double dot_c(int i, double a, double b, double c) {
  double r = 0.0;
  if (cx(i)) r += cx(i) > 0 ? a : -a;
  if (cy(i)) r += cy(i) > 0 ? b : -b;
  if (cz(i)) r += cz(i) > 0 ? c : -c;
  return r;
}

// The thread's node, with consecutive blocks kept on one XCD, and the
// periodic neighbours' byte offsets in an FP64 field (under 2^30: the lattice
// has fewer than 2^31 / 19 nodes); the direction goes into the scalar base of
// a buffer access, so that no access takes vector address arithmetic.
struct Node {
  int id, x, y, z, xs[3], ys[3], zs[3];
  unsigned block;
  bool valid;
  __device__ unsigned off(int dx, int dy, int dz) const {
    return (unsigned)(xs[dx + 1] + ys[dy + 1] + zs[dz + 1]) * 8u;
  }
};
__device__ inline Node node_of(const Geom& g) {
  Node d;
  const int n = (int)g.ncell;
  d.block = xcd_block(blockIdx.x, gridDim.x);
  // (a lane past the lattice takes its last node, stores nothing and adds to
  // no sum)
  const int raw = (int)(d.block * 256u + threadIdx.x);
  d.valid = raw < n;
  d.id = d.valid ? raw : n - 1;
  const int yz = d.id / g.nx;
  d.x = d.id - yz * g.nx;
  d.z = yz / g.ny;
  d.y = yz - d.z * g.ny;
  const int nxy = g.nx * g.ny;
  for (int k = -1; k <= 1; ++k) {
    const int x = d.x + k, y = d.y + k, z = d.z + k;
    d.xs[k + 1] = x < 0 ? g.nx - 1 : (x >= g.nx ? 0 : x);
    d.ys[k + 1] = g.nx * (y < 0 ? g.ny - 1 : (y >= g.ny ? 0 : y));
    d.zs[k + 1] = nxy * (z < 0 ? g.nz - 1 : (z >= g.nz ? 0 : z));
  }
  return d;
}
__device__ inline double load_dir(const double* f, int n, int i, unsigned b) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                        rsrc_of(f + (size_t)i * n), b, 0, 0));
}
__device__ inline void store_dir(double* f, int n, int i, unsigned b, double v) {
  typedef decltype(__builtin_amdgcn_raw_buffer_load_b64(rsrc_of(f), 0, 0, 0)) V;
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), rsrc_of(f + (size_t)i * n), b,
                                        0, 0);
}

// Momentum exchange in reverse, at the nodes owned in o_{t-1}:
//   F_p = -sum S, T_p = -sum r x S,
//   S = sum_i (c_i - u_p) f*_i + (c_i + u_p) f_opp(i)
//     = J* - J_t + u_p (rho_t - rho*)
// with J*, rho* the moments of f*_{t-1} at the node and J_t, rho_t those of
// the streamed f_t.  Sbar = -(Fbar + Tbar x r) goes to dJ/df_t (post-stream
// terms) here and to dJ/df*_{t-1} (own terms) in k_adj_collide, where the
// rest direction's two terms cancel.
// Bound by the latency of its 72 scattered accesses at the owned nodes (a
// tenth of them at 96^3 with 27 cubes): 81 -> 30 us with 32-bit buffer
// addressing and reduce-scatter sums in place of 64-bit index arithmetic and
// twelve full wavefront sums per particle.
__global__ __launch_bounds__(256) void k_adj_mea(const double* __restrict__ fprev,
                                                 double* __restrict__ hbar,
                                                 const int* __restrict__ owner,
                                                 const double* __restrict__ prec,
                                                 const double* __restrict__ fhbar, Geom g,
                                                 double* __restrict__ pbar) {
  const Node d = node_of(g);
  const int n = (int)g.ncell;
  const int o = d.valid ? owner_id(owner[d.id]) : -1;
  double inc[PB];
  for (int k = 0; k < PB; ++k) inc[k] = 0.0;
  if (o >= 0) {
    const unsigned self = (unsigned)d.id * 8u;
    const Exchange e = exchange_at(g, o, d.x, d.y, d.z, prec, fhbar);
    const double sbu = e.Sb[0] * e.up[0] + e.Sb[1] * e.up[1] + e.Sb[2] * e.up[2];
    double dm = 0.0, S[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 1; i < Q; ++i) {
      const double v = load_dir(fprev, n, i, self) -
                       load_dir(fprev, n, i, d.off(-cx(i), -cy(i), -cz(i)));
      dm -= v;
      if (cx(i)) S[0] += cx(i) * v;
      if (cy(i)) S[1] += cy(i) * v;
      if (cz(i)) S[2] += cz(i) * v;
    }
#pragma unroll
    for (int i = 1; i < Q; ++i)
      store_dir(hbar, n, i, self,
                load_dir(hbar, n, i, self) + (sbu - dot_c(i, e.Sb[0], e.Sb[1], e.Sb[2])));
    double upb[3], sxt[3], upxw[3], rxup[3];
    for (int k = 0; k < 3; ++k) {
      S[k] += e.up[k] * dm;
      upb[k] = e.Sb[k] * dm;
    }
    cross(S, e.T, sxt);
    cross(upb, e.W, upxw);
    cross(e.r, upb, rxup);
    for (int k = 0; k < 3; ++k) {
      inc[k] = sxt[k] - upxw[k];    // X
      inc[6 + k] = upb[k];          // U
      inc[9 + k] = rxup[k];         // omega
    }
  }
  commit_adjoint(o, inc, pbar);
}

// Streaming and the own terms of the momentum exchange in reverse,
//   dJ/df*_i(x) = hin_i(x + c_i) + [x owned in o_{t-1}] Sbar . (c_i - u_p),
// then the collision (eqs. (10), (12)-(15)) and the coupling terms of B(d)
// and u_p into the adjoints of P_{t-1}:
//   f* = (1 - w) f + (w - 1) feq(rho, u) + feq(rho, v),  v = u + B (u_p - u) + a
// Bound by its memory traffic: 19 values each of hin, fprev and hout per node
// (404 MB at 96^3).  As one kernel dJ/df* is never written and read back,
// which the collision and the streaming as two did (164 us together at 96^3
// with 27 cubes, 80 us as one).
__global__ __launch_bounds__(256) void k_adj_collide(
    const double* __restrict__ hin, double* __restrict__ hout, const double* __restrict__ fprev,
    const int* __restrict__ owner, const double* __restrict__ prec,
    const double* __restrict__ fhbar, Particles P, Geom g, Phys ph, double* __restrict__ pbar,
    double* __restrict__ abar_part) {
  __shared__ double ared[4][3];
  const Node nd = node_of(g);
  const int n = (int)g.ncell;
  const int o = nd.valid ? owner_id(owner[nd.id]) : -1;

  // moments of f at x
  double rho = 0.0, J[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double f = load_dir(fprev, n, i, nd.off(-cx(i), -cy(i), -cz(i)));
    rho += f;
    if (cx(i)) J[0] += cx(i) * f;
    if (cy(i)) J[1] += cy(i) * f;
    if (cz(i)) J[2] += cz(i) * f;
  }
  // coupling weight and its slope, particle velocity (before dJ/df* is held
  // in registers)
  double B = 0.0, Bp = 0.0, nrm[3] = {0.0, 0.0, 0.0};
  Exchange e = {};
  if (o >= 0) {
    e = exchange_at(g, o, nd.x, nd.y, nd.z, prec, fhbar);
    const double d = sdf_grad(P.shape[o], P.size[o], rec_R(prec + (size_t)PREC_N * o), e.r, nrm,
                              nullptr);
    // B = cos^2(a), dB/dd = -(pi / eps) sin(a) cos(a), a = pi (d + eps/2) / (2 eps)
    B = d <= -0.5 * ph.eps ? 1.0 : 0.0;
    if (d > -0.5 * ph.eps && d < 0.5 * ph.eps) {
      double sn, cs;
      sincospi((d + 0.5 * ph.eps) / (2.0 * ph.eps), &sn, &cs);
      B = cs * cs;
      Bp = -(PI / ph.eps) * (sn * cs);
    }
  }
  // dJ/df* at x
  const double sbu = e.Sb[0] * e.up[0] + e.Sb[1] * e.up[1] + e.Sb[2] * e.up[2];
  double gb[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    gb[i] = load_dir(hin, n, i, nd.off(cx(i), cy(i), cz(i)));
    if (i) gb[i] += dot_c(i, e.Sb[0], e.Sb[1], e.Sb[2]) - sbu;
  }

  // the collision in reverse
  const double u[3] = {J[0] / rho, J[1] / rho, J[2] / rho};
  double v[3];
  for (int k = 0; k < 3; ++k) v[k] = u[k] + B * (e.up[k] - u[k]) + ph.a_ext[k];
  // moments of dJ/df* weighted by w_i: s0, s1 (vector), s2 (symmetric)
  double s0 = 0.0, s1[3] = {0.0, 0.0, 0.0};
  double s2[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double gw = gb[i] * wgt(i);
    const int c[3] = {cx(i), cy(i), cz(i)};
    s0 += gw;
    for (int a = 0; a < 3; ++a) {
      if (c[a]) s1[a] += c[a] * gw;
      for (int b = a; b < 3; ++b)
        if (c[a] * c[b]) s2[a][b] += c[a] * c[b] * gw;
    }
  }
  for (int a = 1; a < 3; ++a)
    for (int b = 0; b < a; ++b) s2[a][b] = s2[b][a];
  // A(w) = d/drho of sum g feq(rho, w); G(w) = d/dw of the same
  auto A = [&](const double* w) {
    double ww = 0.0, s1w = 0.0, wsw = 0.0;
    for (int a = 0; a < 3; ++a) {
      ww += w[a] * w[a];
      s1w += s1[a] * w[a];
      for (int b = 0; b < 3; ++b) wsw += w[a] * s2[a][b] * w[b];
    }
    return s0 + 3.0 * s1w + 4.5 * wsw - 1.5 * ww * s0;
  };
  auto G = [&](const double* w, double* out) {
    for (int a = 0; a < 3; ++a) {
      double sw = 0.0;
      for (int b = 0; b < 3; ++b) sw += s2[a][b] * w[b];
      out[a] = rho * (3.0 * s1[a] + 9.0 * sw - 3.0 * w[a] * s0);
    }
  };
  const double om = ph.omega;
  const double rhob = (om - 1.0) * A(u) + A(v);
  double vb[3], gu[3];
  G(v, vb);
  G(u, gu);
  double ub[3];
  for (int k = 0; k < 3; ++k) ub[k] = ((om - 1.0) * gu[k] + (1.0 - B) * vb[k]) / rho;
  const double rest = rhob - (u[0] * ub[0] + u[1] * ub[1] + u[2] * ub[2]);
  if (nd.valid) {
    const unsigned self = (unsigned)nd.id * 8u;
#pragma unroll
    for (int i = 0; i < Q; ++i)
      store_dir(hout, n, i, self, (1.0 - om) * gb[i] + (rest + dot_c(i, ub[0], ub[1], ub[2])));
  }
  // fluid acceleration adjoint: per-block partial, fixed order
  const bool valid = nd.valid;
  const double a6[6] = {valid ? vb[0] : 0.0, valid ? vb[1] : 0.0, valid ? vb[2] : 0.0,
                        0.0, 0.0, 0.0};
  const double asum = wave_sum6_scatter(a6);
  const int lane = threadIdx.x % WAVE;
  if (lane < 6 && (lane & 1) == 0) ared[threadIdx.x / WAVE][lane >> 1] = asum;
  __syncthreads();
  if (threadIdx.x < 3) {
    const int k = threadIdx.x;
    abar_part[3 * (size_t)nd.block + k] = ((ared[0][k] + ared[1][k]) + ared[2][k]) + ared[3][k];
  }
  double inc[PB];
  for (int k = 0; k < PB; ++k) inc[k] = 0.0;
  if (o >= 0) {
    double Bb = 0.0, upb[3];
    for (int k = 0; k < 3; ++k) {
      Bb += vb[k] * (e.up[k] - u[k]);
      upb[k] = B * vb[k];
    }
    const double db = Bb * Bp;
    double nxr[3], upxw[3], rxup[3];
    cross(nrm, e.r, nxr);
    cross(upb, e.W, upxw);
    cross(e.r, upb, rxup);
    for (int k = 0; k < 3; ++k) {
      inc[k] = -db * nrm[k] - upxw[k];      // X
      inc[3 + k] = db * nxr[k];             // theta
      inc[6 + k] = upb[k];                  // U
      inc[9 + k] = rxup[k];                 // omega
    }
  }
  commit_adjoint(o, inc, pbar);
}

// Particle motion in reverse (eqs. (2)-(3)), one thread per particle:
//   U_t = U + (F_h + F_c)/(s V) + (1 - 1/s) g,   X_t = X + U_t
//   w_t = w + (T_h + T_c)/(s I_1),               R_t = exp([w_t]x) R
// pbar holds Pbar_t; on return it holds Pbar_{t-1} before the node terms, and
// fhbar the adjoints of F_h and T_h (6 per particle).  The fluid acceleration
// of a balanced periodic box, a = -sum (s_p - 1) V_p g / N, adds its s terms:
// every workgroup sums the nblocks partials of its adjoint itself (the same
// order in each), which saves a launch of a single workgroup.
__global__ __launch_bounds__(256) void k_adj_move(Particles P, Phys ph, Geom g, int balance,
                                                  const double* __restrict__ prec_t,
                                                  const double* __restrict__ frc,
                                                  const double* __restrict__ abar_part,
                                                  int nblocks, double* __restrict__ pbar,
                                                  double* __restrict__ fhbar,
                                                  double* __restrict__ sbar) {
  __shared__ double red[4][3];
  double abar[3] = {0.0, 0.0, 0.0};
  if (balance) {
    for (int b = threadIdx.x; b < nblocks; b += 256)
      for (int k = 0; k < 3; ++k) abar[k] += abar_part[3 * (size_t)b + k];
    for (int k = 0; k < 3; ++k) {
      const double t = wave_sum(abar[k]);
      if (threadIdx.x % WAVE == 0) red[threadIdx.x / WAVE][k] = t;
    }
    __syncthreads();
    for (int k = 0; k < 3; ++k) abar[k] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
  }
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= P.n) return;
  double* pb = pbar + PB * p;
  const double s = P.dens[p], V = P.vol[p];
  const double I1 = P.inert[p] / s;
  const double* f = frc + 12 * p;       // Fh 3, Th 3, Fc 3, Tc 3
  const double* W = rec_W(prec_t + (size_t)PREC_N * p);
  double Xb[3], thb[3], Ub[3], Wb[3];
  for (int k = 0; k < 3; ++k) {
    Xb[k] = pb[k];
    thb[k] = pb[3 + k];
    Ub[k] = pb[6 + k] + pb[k];          // X_t = X + U_t
    Wb[k] = pb[9 + k];
  }
  // rotation: R_t = E R_{t-1} with E = exp([w_t]x)
  const double th2 = W[0] * W[0] + W[1] * W[1] + W[2] * W[2];
  const double th = sqrt(th2);
  double a, b, sa, ca;
  if (th < 1e-4) {
    a = 0.5 - th2 / 24.0;
    b = 1.0 / 6.0 - th2 / 120.0;
  } else {
    a = (1.0 - cos(th)) / th2;
    b = (th - sin(th)) / (th2 * th);
  }
  sa = th < 1e-4 ? 1.0 - th2 / 6.0 : sin(th) / th;
  ca = a;   // (1 - cos)/th^2
  // E^T v = v - sa (w x v) + ca w x (w x v)
  double wxt[3], wwxt[3];
  cross(W, thb, wxt);
  cross(W, wxt, wwxt);
  double thb_prev[3], jt[3];
  for (int k = 0; k < 3; ++k) {
    thb_prev[k] = thb[k] - sa * wxt[k] + ca * wwxt[k];
    jt[k] = thb[k] - a * wxt[k] + b * wwxt[k];   // J_l(w)^T thb
  }
  for (int k = 0; k < 3; ++k) Wb[k] += jt[k];
  double ds = 0.0;
  for (int k = 0; k < 3; ++k) {
    ds += Ub[k] * (-(f[k] + f[6 + k]) / (s * s * V) + ph.gravity[k] / (s * s));
    ds += Wb[k] * (-(f[3 + k] + f[9 + k]) / (s * s * I1));
  }
  if (balance)
    for (int k = 0; k < 3; ++k) ds += abar[k] * (-V * ph.gravity[k] / (double)g.ncell);
  sbar[p] += ds;
  for (int k = 0; k < 3; ++k) {
    fhbar[6 * p + k] = Ub[k] / (s * V);
    fhbar[6 * p + 3 + k] = Wb[k] / (s * I1);
    pb[k] = Xb[k];
    pb[3 + k] = thb_prev[k];
    pb[6 + k] = Ub[k];
    pb[9 + k] = Wb[k];
  }
}

// Copy the particle state (X, q, U, W, R) into a record array and, after a
// step (frc given), the step's forces (F_h, T_h, F_c, T_c) into another.
__global__ void k_record(Particles P, const double* Fh, const double* Th, const double* Fc,
                         const double* Tc, double* __restrict__ prec, double* __restrict__ frc) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P.n) return;
  double* r = prec + (size_t)PREC_N * p;
  for (int k = 0; k < 3; ++k) r[k] = P.X[3 * p + k];
  for (int k = 0; k < 4; ++k) r[3 + k] = P.q[4 * p + k];
  for (int k = 0; k < 3; ++k) r[7 + k] = P.U[3 * p + k];
  for (int k = 0; k < 3; ++k) r[10 + k] = P.W[3 * p + k];
  for (int k = 0; k < 9; ++k) r[13 + k] = P.R[9 * p + k];
  if (!frc) return;
  for (int k = 0; k < 3; ++k) {
    frc[12 * p + k] = Fh[3 * p + k];
    frc[12 * p + 3 + k] = Th[3 * p + k];
    frc[12 * p + 6 + k] = Fc[3 * p + k];
    frc[12 * p + 9 + k] = Tc[3 * p + k];
  }
}

__global__ void k_fill_zero(double* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

int adjoint_record_doubles() { return PREC_N; }
int adjoint_slots() { return PB; }

hipError_t launch_record(Ctx& c, double* prec, double* frc) {
  if (c.np == 0) return hipSuccess;
  hipLaunchKernelGGL(k_record, dim3(nblk(c.np)), dim3(256), 0, c.stream, c.part, c.Fh, c.Th,
                     c.Fc, c.Tc, prec, frc);
  return hipGetLastError();
}

hipError_t launch_fill_zero(Ctx& c, double* p, long long n) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_zero, dim3(nblk(n)), dim3(256), 0, c.stream, p, n);
  return hipGetLastError();
}

// work: the adjoints of F_h, T_h (6 np), then the per-block partials of the
// fluid acceleration's adjoint (3 per workgroup of k_adj_collide)
hipError_t launch_adjoint_move(Ctx& c, const double* prec, const double* frc, double* pbar,
                               double* sbar, double* work) {
  if (c.np == 0) return hipSuccess;
  double* fhbar = work;
  double* apart = work + 6 * (size_t)c.np;
  hipLaunchKernelGGL(k_adj_move, dim3(nblk(c.np)), dim3(256), 0, c.stream, c.part, c.ph, c.g,
                     c.P.balance ? 1 : 0, prec, frc, apart, (int)nblk(c.g.ncell), pbar, fhbar,
                     sbar);
  return hipGetLastError();
}

hipError_t launch_adjoint_node(Ctx& c, double* hin, double* hout, const double* fown,
                               const double* fprev, const int* owner, const double* prec,
                               double* pbar, double* work) {
  double* fhbar = work;
  double* apart = work + 6 * (size_t)c.np;
  const dim3 nb(nblk(c.g.ncell)), nt(256);
  hipLaunchKernelGGL(k_adj_mea, nb, nt, 0, c.stream, fown, hin, owner, prec, fhbar, c.g, pbar);
  if (hout)
    hipLaunchKernelGGL(k_adj_collide, nb, nt, 0, c.stream, hin, hout, fprev, owner, prec, fhbar,
                       c.part, c.g, c.ph, pbar, apart);
  return hipGetLastError();
}

size_t adjoint_work_doubles(const Ctx& c) {
  return 6 * (size_t)c.np + 3 * (size_t)nblk(c.g.ncell);
}

}  // namespace hlbm
