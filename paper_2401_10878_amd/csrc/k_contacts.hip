// Discrete contact treatment (Sec. 3.3.1, eqs. (4)-(9)) and the clearing of
// the pair tables and counters outside the steps.
//
// One workgroup treats one contact record (the workgroups of a fixed grid
// take the table's occupied slots from its list in a stride):
//   box      the carried (corrected) box of an established contact, or the
//            rough box [min - 1/2, max + 1/2] of the flagged node images;
//            kept in the frame of the lower-id particle a (Sec. 3.3.2)
//   correct  faces -x,+x,-y,+y,-z,+z in turn; N_c x N_c midpoint samples of
//            phi = max(d'_a, d'_b) on the face; the face moves inwards by
//            the minimum of phi
//   integrate N_c^3 midpoint samples of the box; inside = both enlarged
//            distances negative; sums of count, position and gradient
//            difference, maximum of -(d'_a + d'_b)
//   force    normal force (4, 5, 6) and friction (7-9) at the centroid,
//            appended to both particles' contact slots; k_particles sums a
//            particle's slots in the order of the partner id, so the
//            result does not depend on the order the pairs ran in.
#include <float.h>

#include "balance.h"
#include "context.h"

namespace hlbm {

namespace {

// Tile counts (CLEAR_TILES) and, once after allocation, every slot of a
// table (CLEAR_ALL_SLOTS), over a grid.
__global__ void k_clear_grid(PairTable table, int* dcount, long long ndt, int* lcount,
                             long long nlt, int what) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long stride = (long long)gridDim.x * blockDim.x;
  if (what & CLEAR_TILES) {
    for (long long i = tid; i < ndt; i += stride) dcount[i] = 0;
    for (long long i = tid; i < nlt; i += stride) lcount[i] = 0;
  }
  if (what & CLEAR_ALL_SLOTS)
    for (long long i = tid; i < table.cap; i += stride) clear_slot(table, i);
}

// The slots a table's list names and the particles' contact slots
// (CLEAR_TABLE), the contact forces and the sample counter (CLEAR_RESULTS),
// one workgroup: the list count is reset after the workgroup barrier, when every
// thread has read it.
constexpr int CLEAR_THREADS = 1024;
__global__ __launch_bounds__(CLEAR_THREADS) void k_clear_state(PairTable table, double* Fc,
                                                               double* Tc, int np, int* ccount,
                                                               Counters* ctr, int what) {
  const int tid = (int)threadIdx.x;
  if (what & CLEAR_TABLE) {
    const int nl = *table.nlist;
    for (int i = tid; i < nl; i += CLEAR_THREADS) {
      const int s = table.list[i];
      if (what & CLEAR_COUNT)
        atomicAdd(&ctr->total_cells, (unsigned long long)table.rec[s].count);
      clear_slot(table, s);
    }
    for (int i = tid; i < np; i += CLEAR_THREADS) ccount[i] = 0;
  }
  if (what & CLEAR_RESULTS) {
    for (long long i = tid; i < 3LL * np; i += CLEAR_THREADS) {
      Fc[i] = 0.0;
      Tc[i] = 0.0;
    }
    if (tid == 0) ctr->samples = 0;
  }
  __syncthreads();
  if (tid == 0) {
    if (what & CLEAR_TABLE) *table.nlist = 0;
  }
}

__global__ __launch_bounds__(CLEAR_THREADS) void k_count(PairTable table, Counters* ctr) {
  __shared__ unsigned long long sum[2];
  if (threadIdx.x == 0) sum[0] = sum[1] = 0;
  __syncthreads();
  const int n = *table.nlist;
  unsigned long long pairs = 0, cells = 0;
  for (int i = (int)threadIdx.x; i < n; i += CLEAR_THREADS) {
    const int c = table.rec[table.list[i]].count;
    pairs += c > 0 ? 1 : 0;
    cells += (unsigned)c;
  }
  if (pairs) {
    atomicAdd(&sum[0], pairs);
    atomicAdd(&sum[1], cells);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    ctr->det_pairs = sum[0];
    ctr->det_cells = sum[1];
  }
}

struct Body {
  int shape;
  double size, X[3], R[9];
};

// Signed distance of the member that a wavefront evaluates, its enlargement
// taken off (particle), or the distance to the wall plane (-1 bottom, -2
// top).  With a gradient, a point farther outside a polyhedron than far may
// return a lower bound (far = delta: only points inside the enlarged body
// need the exact value and gradient).
template <bool ELL>
__device__ inline double member_sdf(const Body& b, int id, const PolyDev* poly, double delta,
                                    double nz, const double* y, double* g,
                                    double far = 1e300) {
  if (id >= 0) {
    const double r[3] = {y[0] - b.X[0], y[1] - b.X[1], y[2] - b.X[2]};
    if (g) return sdf_grad_exact<ELL>(b.shape, b.size, b.R, r, g, poly, far) - delta;
    return sdf_exact<ELL>(b.shape, b.size, b.R, r[0], r[1], r[2], poly) - delta;
  }
  if (g) {
    g[0] = 0.0;
    g[1] = 0.0;
    g[2] = id == -1 ? 1.0 : -1.0;
  }
  return id == -1 ? y[2] + 0.5 : (nz - 0.5) - y[2];
}

__device__ inline void cross3(const double* a, const double* b, double* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}

// Append (force, torque) on particle p from its partner `other` to p's slots.
__device__ void add_contact(Tiles tl, Counters* ctr, int p, int other,
                            const double* F, const double* T) {
  const int k = atomicAdd(&tl.ccount[p], 1);
  if (k >= MAXC) {
    atomicOr(&ctr->contact_overflow, 1);
    return;
  }
  const size_t e = (size_t)p * MAXC + k;
  tl.ckey[e] = other;
  for (int m = 0; m < 3; ++m) {
    tl.cval[6 * e + m] = F[m];
    tl.cval[6 * e + 3 + m] = T[m];
  }
}

// One workgroup of four wavefronts per record: wavefronts 0 and 1 evaluate
// the first member's distance, 2 and 3 the second's, 128 samples at a time,
// and exchange them through LDS.  The treatment of a record is a chain of
// dependent evaluations (three axes, then the integration samples of a lane)
// and not a matter of throughput: two bodies at once, both faces of an axis
// at once and 128 samples a round leave 7 single evaluations in the chain at
// n_c = 8 where one wavefront per record had 28, and the rolled loop over the
// axes (coordinates by selects) keeps one copy of the distance in the
// instruction cache instead of twelve.  256^3 with 1834 cubes, us: 22.7; one face
// at a time 25.5, eight wavefronts per record 45.3.  Every wavefront forms the
// same minima and sums, so the box corrections and exits are uniform over the
// workgroup; wavefront 0 forms the forces.
constexpr int TREAT_WAVES = 4;
constexpr int TREAT_HALF = TREAT_WAVES / 2;    // wavefronts per member
constexpr int TREAT_ROUND = TREAT_HALF * WAVE;   // samples evaluated between two barriers
struct TreatShared {
  double d[2][2][TREAT_ROUND];     // [round parity][member][sample]
  double red[TREAT_WAVES][8];      // sums of the integration per wavefront
};

template <bool POLY, bool ELL>
__device__ void treat_slot(const PairTable& t, const Particles& P, const Geom& g,
                           const Phys& ph, const FastDiv& fnc, const Tiles& tl, Counters* ctr,
                           int slot, TreatShared& sh, int& round) {
  const int lane = threadIdx.x % WAVE;
  const int wave = (int)((unsigned)__builtin_amdgcn_readfirstlane(threadIdx.x) / WAVE);
  const int member = wave / TREAT_HALF;           // 0: particle a, 1: particle or wall b
  const int at = (wave % TREAT_HALF) * WAVE + lane;   // sample of a round
  PairRec* rec = &t.rec[slot];
  const int a = __builtin_amdgcn_readfirstlane(rec->a);
  const int b = __builtin_amdgcn_readfirstlane(rec->b);
  const bool carried = rec->carried != 0;
  const bool perz = g.periodic_z != 0;
  const double L[3] = {(double)g.nx, (double)g.ny, (double)g.nz};
  const bool per[3] = {true, true, perz};
  const int nc = ph.n_c;
  const double delta = ph.delta_c;
  const PolyDev* poly = POLY ? P.poly : nullptr;

  double XA[3];
  for (int k = 0; k < 3; ++k) XA[k] = P.X[3 * a + k];
  const int id = member == 0 ? a : b;
  Body M;
  M.shape = 0;
  M.size = 0.0;
  for (int k = 0; k < 3; ++k) M.X[k] = 0.0;
  for (int k = 0; k < 9; ++k) M.R[k] = 0.0;
  if (id >= 0) {
    M.shape = P.shape[id];
    M.size = P.size[id];
    // the higher-id particle is moved next to the lower-id one
    for (int k = 0; k < 3; ++k)
      M.X[k] = member == 0 ? XA[k] : XA[k] + minimg(P.X[3 * id + k] - XA[k], L[k], per[k]);
    for (int k = 0; k < 9; ++k) M.R[k] = P.R[9 * id + k];
  }

  double lo[3], hi[3];
  // a new particle-wall pair: the flagged nodes lie on the fluid side of
  // the wall plane and the overlap beyond it, so the wall-side face starts
  // at the far side of the enlarged body (half extent along z plus the
  // enlargement) and the correction moves it onto the body
  double wall_lo = 1e300, wall_hi = -1e300;
  if (!carried && b < 0) {
    const double ez = half_extent(P.shape[a], P.size[a], P.R + 9 * a, 2, poly) + delta;
    if (b == -1) wall_lo = XA[2] - ez;
    else wall_hi = XA[2] + ez;
  }
  for (int k = 0; k < 3; ++k) {
    lo[k] = carried ? rec->lo[k] : (double)rec->rlo[k] - 0.5;
    hi[k] = carried ? rec->hi[k] : (double)rec->rhi[k] + 0.5;
    if (k == 2) {
      lo[k] = fmin(lo[k], wall_lo);
      hi[k] = fmax(hi[k], wall_hi);
    }
    const double mid = 0.5 * (lo[k] + hi[k]);
    const int sh = image_shift(mid - XA[k], L[k], per[k]);
    lo[k] += (double)(sh * (int)L[k]);
    hi[k] += (double)(sh * (int)L[k]);
  }

  // ---- box correction, one pass -----------------------------------------
  bool ok = true;
  int nfaces = 0;   // faces sampled (the box can empty on the way)
  const int nn = nc * nc;
#pragma unroll 1
  for (int k = 0; k < 3; ++k) {
    ok = ok && hi[0] > lo[0] && hi[1] > lo[1] && hi[2] > lo[2];
    if (!ok) break;
    ++nfaces;
    // the two faces of an axis together: the correction of the lower moves
    // no sample of the upper (samples 0 .. nn-1 and nn .. 2 nn-1)
    const double h0 = (hi[0] - lo[0]) / (double)nc, h1 = (hi[1] - lo[1]) / (double)nc,
                 h2 = (hi[2] - lo[2]) / (double)nc;
    double smin = DBL_MAX, smax = DBL_MAX;        // of the lower, of the upper face
#pragma unroll 1
    for (int base = 0; base < 2 * nn; base += TREAT_ROUND) {
      double (*d)[TREAT_ROUND] = sh.d[round & 1];
      ++round;
      if (base + at < 2 * nn) {
        const bool plus = base + at >= nn;
        const int idx = base + at - (plus ? nn : 0);
        // sample (j, l) of the face: j along the first of its two axes
        const int j = (int)fdiv((unsigned)idx, fnc), l = idx - j * nc;
        const double sj = (double)j + 0.5, sl = (double)l + 0.5;
        double y[3];
        y[0] = k == 0 ? (plus ? hi[0] : lo[0]) : lo[0] + sj * h0;
        y[1] = k == 1 ? (plus ? hi[1] : lo[1]) : lo[1] + (k == 0 ? sj : sl) * h1;
        y[2] = k == 2 ? (plus ? hi[2] : lo[2]) : lo[2] + sl * h2;
        d[member][at] = member_sdf<ELL>(M, id, poly, delta, L[2], y, nullptr);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < TREAT_ROUND; u += WAVE) {
        const int i = base + u + lane;
        if (i < 2 * nn) {
          const double m = fmax(d[0][u + lane], d[1][u + lane]);
          if (i < nn) smin = fmin(smin, m);
          else smax = fmin(smax, m);
        }
      }
    }
    smin = wave_min(smin);
    smax = wave_min(smax);
    for (int m = 0; m < 3; ++m) lo[m] = k == m ? lo[m] + smin : lo[m];
    ok = ok && hi[0] > lo[0] && hi[1] > lo[1] && hi[2] > lo[2];
    if (!ok) break;
    ++nfaces;
    for (int m = 0; m < 3; ++m) hi[m] = k == m ? hi[m] - smax : hi[m];
  }
  ok = ok && hi[0] > lo[0] && hi[1] > lo[1] && hi[2] > lo[2];
  // midpoint samples of this record (each evaluates both members)
  if (threadIdx.x == 0) rec->samples = nfaces * nc * nc + (ok ? nc * nc * nc : 0);

  // ---- overlap integration ------------------------------------------------
  int n_in = 0;
  double sy[3] = {0.0, 0.0, 0.0}, gs[3] = {0.0, 0.0, 0.0};
  double dmax = -DBL_MAX;
  double h[3] = {0.0, 0.0, 0.0};
  if (ok) {
    for (int k = 0; k < 3; ++k) h[k] = (hi[k] - lo[k]) / (double)nc;
    const int ns = nc * nc * nc;
#pragma unroll 1
    for (int base = 0; base < ns; base += TREAT_ROUND) {
      double (*d)[TREAT_ROUND] = sh.d[round & 1];
      ++round;
      const int idx = base + at;
      double y[3] = {0.0, 0.0, 0.0}, gr[3] = {0.0, 0.0, 0.0};
      if (idx < ns) {
        const int q = (int)fdiv((unsigned)idx, fnc), l = (int)fdiv((unsigned)q, fnc);
        const int j = idx - q * nc, kk = q - l * nc;
        y[0] = lo[0] + ((double)j + 0.5) * h[0];
        y[1] = lo[1] + ((double)kk + 0.5) * h[1];
        y[2] = lo[2] + ((double)l + 0.5) * h[2];
        // a sample counts when inside both enlarged bodies: beyond delta
        // outside either, a lower bound decides.  A body type's gradient
        // comes with its distance; the built-in shapes' takes divisions and
        // is formed below, for counted samples only
        d[member][at] = member_sdf<ELL>(M, id, poly, delta, L[2], y, POLY ? gr : nullptr, delta);
      }
      __syncthreads();
      const double da = d[0][at], db = d[1][at];
      if (idx < ns && fmax(da, db) < 0.0) {
        if (!POLY) member_sdf<ELL>(M, id, poly, delta, L[2], y, gr, delta);
        for (int m = 0; m < 3; ++m) gs[m] += member == 0 ? gr[m] : -gr[m];
        n_in++;
        dmax = fmax(dmax, -(da + db));
        for (int m = 0; m < 3; ++m) sy[m] += y[m];
      }
    }
    // the wavefronts of both members hold the same samples: counts,
    // positions and depths from the first member's, gradients from all
    const double v[8] = {(double)wave_sum_i(n_in), wave_max(dmax), wave_sum(sy[0]),
                         wave_sum(sy[1]),          wave_sum(sy[2]), wave_sum(gs[0]),
                         wave_sum(gs[1]),          wave_sum(gs[2])};
    if (lane == 0)
      for (int k = 0; k < 8; ++k) sh.red[wave][k] = v[k];
    __syncthreads();
    double w[8];
    for (int k = 0; k < 8; ++k) {
      w[k] = sh.red[0][k];
      for (int i = 1; i < (k < 5 ? TREAT_HALF : TREAT_WAVES); ++i)
        w[k] = k == 1 ? fmax(w[k], sh.red[i][k]) : w[k] + sh.red[i][k];
    }
    n_in = (int)w[0];
    dmax = w[1];
    for (int m = 0; m < 3; ++m) {
      sy[m] = w[2 + m];
      gs[m] = w[5 + m];
    }
  }
  // (the other wavefronts go on to the next record; they write sh.red only
  // after barriers that wavefront 0 reaches once it is done with this one)
  if (wave != 0) return;
  if (!ok || n_in == 0) {
    if (lane == 0) {
      rec->keep = 0;
      rec->n_in = 0;
      rec->volume = 0.0;
    }
    return;
  }

  // ---- results and forces (wave-uniform values) ----------------------------
  double XB[3] = {0.0, 0.0, 0.0};
  if (b >= 0)
    for (int k = 0; k < 3; ++k)
      XB[k] = XA[k] + minimg(P.X[3 * b + k] - XA[k], L[k], per[k]);
  const double V = (double)n_in * (h[0] * h[1] * h[2]);
  double xc[3], nrm[3] = {0.0, 0.0, 0.0};
  for (int m = 0; m < 3; ++m) xc[m] = sy[m] / (double)n_in;
  const double gn = sqrt(gs[0] * gs[0] + gs[1] * gs[1] + gs[2] * gs[2]);
  if (gn > 0.0) {
    for (int m = 0; m < 3; ++m) nrm[m] = gs[m] / gn;
  } else {
    double dv[3];
    if (b >= 0) {
      for (int m = 0; m < 3; ++m) dv[m] = XB[m] - XA[m];
    } else {
      dv[0] = 0.0; dv[1] = 0.0; dv[2] = b == -1 ? -1.0 : 1.0;
    }
    const double dn = sqrt(dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2]);
    if (dn > 0.0)
      for (int m = 0; m < 3; ++m) nrm[m] = dv[m] / dn;
  }
  const double depth = dmax;

  double ra[3], t3[3], va[3], vb[3] = {0.0, 0.0, 0.0};
  for (int m = 0; m < 3; ++m) ra[m] = xc[m] - XA[m];
  cross3(P.W + 3 * a, ra, t3);
  for (int m = 0; m < 3; ++m) va[m] = P.U[3 * a + m] + t3[m];
  double rb[3] = {0.0, 0.0, 0.0};
  if (b >= 0) {
    for (int m = 0; m < 3; ++m) rb[m] = xc[m] - XB[m];
    cross3(P.W + 3 * b, rb, t3);
    for (int m = 0; m < 3; ++m) vb[m] = P.U[3 * b + m] + t3[m];
  }
  double v[3];
  for (int m = 0; m < 3; ++m) v[m] = va[m] - vb[m];
  const double dn = v[0] * nrm[0] + v[1] * nrm[1] + v[2] * nrm[2];
  int established = rec->established;
  double damping = rec->damping;
  if (!established) {
    const double e = ph.restitution;
    damping = dn > 0.0 ? 1.5 * (1.0 - e) * (11.0 - e) / ((1.0 + 9.0 * e) * dn) : 0.0;
    established = 1;
  }
  double fn = 4.0 / (3.0 * PI) * ph.estar * sqrt(V * depth) * (1.0 + damping * dn);
  if (fn < 0.0) fn = 0.0;
  double vt[3];
  for (int m = 0; m < 3; ++m) vt[m] = v[m] - dn * nrm[m];
  const double vtn = sqrt(vt[0] * vt[0] + vt[1] * vt[1] + vt[2] * vt[2]);
  double ft[3] = {0.0, 0.0, 0.0};
  if (vtn > 0.0) {
    const double aa = vtn / ph.u_k;
    const double rr = ph.mu_k / ph.mu_s;
    const double mus = ph.mu_s * (1.0 - 0.09 * (rr * rr * rr * rr));
    const double a2 = aa * aa;
    const double mu = (2.0 * mus - ph.mu_k) * a2 / (a2 * a2 + 1.0) + ph.mu_k -
                      ph.mu_k / (a2 + 1.0);
    for (int m = 0; m < 3; ++m) ft[m] = -(vt[m] / vtn) * mu * fn;
  }
  double Fa[3], Ta[3], Tb[3];
  for (int m = 0; m < 3; ++m) Fa[m] = -fn * nrm[m] + ft[m];
  cross3(ra, Fa, Ta);
  // lane 0 appends to particle a, lane 1 to particle b: one round trip of
  // the slot counts
  if (lane < (b >= 0 ? 2 : 1)) {
    double F[3], T[3];
    const double Fb[3] = {-Fa[0], -Fa[1], -Fa[2]};
    cross3(rb, Fb, Tb);
    for (int m = 0; m < 3; ++m) {
      F[m] = lane == 0 ? Fa[m] : Fb[m];
      T[m] = lane == 0 ? Ta[m] : Tb[m];
    }
    add_contact(tl, ctr, lane == 0 ? a : b, lane == 0 ? b : a, F, T);
  }
  if (lane == 0) {
    rec->keep = 1;
    rec->carried = 1;
    rec->established = established;
    rec->damping = damping;
    rec->age = rec->age + 1;
    rec->n_in = n_in;
    rec->volume = V;
    rec->depth = depth;
    rec->fn = fn;
    for (int m = 0; m < 3; ++m) {
      rec->lo[m] = lo[m];
      rec->hi[m] = hi[m];
      rec->centroid[m] = xc[m];
      rec->normal[m] = nrm[m];
      rec->force_a[m] = Fa[m];
    }
  }
}

constexpr int TREAT_BLOCKS = 1024;
template <bool POLY, bool ELL = false>
__global__ __launch_bounds__(TREAT_WAVES* WAVE) void k_treat(PairTable t, Particles P, Geom g,
                                                             Phys ph, FastDiv fnc, Tiles tl,
                                                             Counters* ctr, int* next_nlist,
                                                             unsigned blocks,
                                                             const double* __restrict__ bal_part,
                                                             unsigned bal_blocks,
                                                             double* __restrict__ bal_out) {
  if (blockIdx.x >= blocks) {
    // workgroups past the treatment's: the first stage of the balance sums
    balance_stage1(bal_part, bal_blocks,
                   (blockIdx.x - blocks) * TREAT_WAVES + threadIdx.x / WAVE, bal_out);
    return;
  }
  __shared__ TreatShared sh;
  const int n = *t.nlist;
  int round = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *next_nlist = 0;
    ctr->samples = 0;
  }
  for (int i = (int)blockIdx.x; i < n; i += (int)blocks)
    treat_slot<POLY, ELL>(t, P, g, ph, fnc, tl, ctr,
                          __builtin_amdgcn_readfirstlane(t.list[i]), sh, round);
}

}  // namespace

hipError_t launch_clear(Ctx& c, PairTable table, int what) {
  const long long ndt = (long long)c.g.dtx * c.g.dty * c.g.dtz;
  const long long nlt = (long long)c.g.ltx * c.g.lty * c.g.ltz;
  if (what & (CLEAR_TILES | CLEAR_ALL_SLOTS)) {
    long long work = (what & CLEAR_ALL_SLOTS) ? table.cap : 0;
    if ((what & CLEAR_TILES) && ndt > work) work = ndt;
    long long blocks = (work + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_clear_grid, dim3((unsigned)blocks), dim3(256), 0, c.stream, table,
                       c.tl.dcount, ndt, c.tl.lcount, nlt, what);
  }
  if (what & (CLEAR_TABLE | CLEAR_RESULTS))
    hipLaunchKernelGGL(k_clear_state, dim3(1), dim3(CLEAR_THREADS), 0, c.stream, table, c.Fc,
                       c.Tc, c.np, c.tl.ccount, c.counters, what);
  return hipGetLastError();
}

hipError_t launch_count(Ctx& c, PairTable table) {
  hipLaunchKernelGGL(k_count, dim3(1), dim3(CLEAR_THREADS), 0, c.stream, table, c.counters);
  return hipGetLastError();
}

hipError_t launch_treat(Ctx& c, PairTable t, PairTable next, bool balance) {
  const unsigned blocks = (unsigned)(t.cap < TREAT_BLOCKS ? t.cap : TREAT_BLOCKS);
  const dim3 nb(blocks + (balance ? BAL_PARTS / TREAT_WAVES : 0)), nt(TREAT_WAVES * WAVE);
  const FastDiv fnc = make_fastdiv((unsigned)c.ph.n_c);
  const unsigned nlt = (unsigned)c.g.ltx * (unsigned)c.g.lty * (unsigned)c.g.ltz;
  auto k = c.has_ellipsoid ? k_treat<true, true> : (c.has_poly ? k_treat<true> : k_treat<false>);
  hipLaunchKernelGGL(k, nb, nt, 0, c.stream, t, c.part, c.g, c.ph, fnc, c.tl, c.counters,
                     next.nlist, blocks, c.bal_part, nlt,
                     c.bal_part ? c.bal_part + 4 * (size_t)nlt : nullptr);
  return hipGetLastError();
}

}  // namespace hlbm
