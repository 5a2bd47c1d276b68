// Host-side context of the library and the launch interface of each kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <string>

#include "../../include/hlbm.h"
#include "device_math.h"

namespace hlbm {

// One contact-pair record of the open-addressing pair table.  count, rlo and
// rhi are written with atomics by the rough detection; the rest is written
// by the single wavefront that treats the record, or by the copy that
// carries a kept contact into the next step's table.
struct PairRec {
  int a, b;
  int count;
  int rlo[3], rhi[3];
  int carried, established, age, n_in, keep;
  int samples;   // midpoint samples of the latest treatment
  double lo[3], hi[3];
  double damping;
  double volume, centroid[3], normal[3], depth, fn, force_a[3];
};

struct PairTable {
  uint64_t* keys;   // [cap], EMPTY_KEY when free
  PairRec* rec;     // [cap]
  int cap;          // power of two
  // the occupied slots in order of insertion (list[0 .. *nlist)), so that
  // the treatment and the clearing visit only those; both follow the keys
  // in one allocation (key_block_bytes) and are copied with them
  int* list;
  int* nlist;
};
inline size_t key_block_bytes(int cap) {
  return sizeof(uint64_t) * (size_t)cap + sizeof(int) * ((size_t)cap + 2);
}
inline void set_table_views(PairTable& t) {
  t.list = (int*)(t.keys + t.cap);
  t.nlist = t.list + t.cap;
}
// A key inserted into slot h (by the inserting thread only) joins the list.
__device__ inline void list_slot(const PairTable& t, uint32_t h) {
  t.list[atomicAdd(t.nlist, 1)] = (int)h;
}

// Device counters and flags (one small block of device memory).
struct Counters {
  // keys with count > 0 and sum of their counts, latest detection: formed
  // from the records when asked for (launch_count)
  unsigned long long det_pairs;
  unsigned long long det_cells;
  unsigned long long total_cells;  // sum over the detections before the latest
  unsigned long long steps;
  // midpoint samples of the latest treatment (reset by it, summed by the
  // carry-over that follows it)
  unsigned long long samples;
  int tile_overflow;
  int pair_overflow;
  int unstable;
  int contact_overflow;   // more than MAXC contacts on one particle
  // zero-net-flux balance force (balance mode 2): controller part b of the
  // fluid acceleration, lattice momentum P after the last collision,
  // lattice mass M, and the acceleration a = fluid_accel + b in use
  double bal_b[3], bal_P[3], bal_M, bal_a[3];
};

// Three values per thread of a 256-thread workgroup, stored as consecutive
// triples from out[3 * first] on, limited to n triples: through LDS, so that
// the lanes write consecutive words (the target is host memory, where every
// partial line is a transaction of its own).
__device__ inline void store_rows3(double* sh, const double* v, long long first, long long n,
                                   double* out) {
  for (int k = 0; k < 3; ++k) sh[3 * threadIdx.x + k] = v[k];
  __syncthreads();
  for (int k = 0; k < 3; ++k) {
    const long long i = 3 * first + k * 256 + (int)threadIdx.x;
    if (i < 3 * n) out[i] = sh[k * 256 + threadIdx.x];
  }
}

__device__ inline void clear_slot(const PairTable& t, long long i) {
  t.keys[i] = EMPTY_KEY;
  PairRec r = {};
  for (int k = 0; k < 3; ++k) {
    r.rlo[k] = 0x7fffffff;
    r.rhi[k] = (int)0x80000000;
  }
  t.rec[i] = r;
}

// Carry-over of occupied slot s of the pair table `from` into `to` when its
// record is marked to be kept (an established contact that continues, Sec.
// 3.3.2): the key is inserted by linear probing and the record's contact
// state copied; a full table raises pair_overflow.
__device__ inline void keep_slot(const PairTable& from, const PairTable& to, long long s,
                                 Counters* ctr) {
  const uint64_t key = from.keys[s];
  const PairRec& r = from.rec[s];
  if (!r.keep) return;
  const uint32_t mask = (uint32_t)to.cap - 1u;
  uint32_t h = pair_hash(key) & mask;
  for (int probe = 0; probe < to.cap; ++probe) {
    unsigned long long old = atomicCAS((unsigned long long*)&to.keys[h],
                                       (unsigned long long)EMPTY_KEY,
                                       (unsigned long long)key);
    if (old == EMPTY_KEY) list_slot(to, h);
    if (old == EMPTY_KEY || old == key) {
      PairRec& d = to.rec[h];
      d.a = r.a;
      d.b = r.b;
      d.carried = 1;
      d.established = r.established;
      d.age = r.age;
      d.n_in = r.n_in;
      d.keep = 0;
      for (int k = 0; k < 3; ++k) {
        d.lo[k] = r.lo[k];
        d.hi[k] = r.hi[k];
        d.centroid[k] = r.centroid[k];
        d.normal[k] = r.normal[k];
        d.force_a[k] = r.force_a[k];
      }
      d.damping = r.damping;
      d.volume = r.volume;
      d.depth = r.depth;
      d.fn = r.fn;
      return;
    }
    h = (h + 1u) & mask;
  }
  atomicOr(&ctr->pair_overflow, 1);
}

// Division of 0 <= n < 2^31 by a fixed divisor d >= 1 with one multiply-high
// and a shift (Granlund and Montgomery, PLDI 1994): with s = ceil(log2 d)
// and m = floor(2^32 (2^s - d) / d) + 1, n / d = (mulhi(n, m) + n) >> s; the
// sum stays below 2^32 because mulhi(n, m) <= n.
struct FastDiv {
  unsigned d, m, s;
};
inline FastDiv make_fastdiv(unsigned d) {
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  const unsigned long long m = ((1ull << 32) * ((1ull << s) - d)) / d + 1;
  return FastDiv{d, (unsigned)m, s};
}
__host__ __device__ inline unsigned fdiv(unsigned n, FastDiv f) {
  return (unsigned)(((((unsigned long long)n * f.m) >> 32) + n) >> f.s);
}

// Loads and stores at byte offset b of an array as raw buffer operations: a
// scalar resource over the array from p (no range check is relied on; every
// offset lies inside the array) and a 32-bit per-lane byte offset, which the
// hardware adds without vector address arithmetic.
__device__ inline __amdgpu_buffer_rsrc_t rsrc_of(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00020000);
}
// Logical block id with consecutive ids kept on one XCD (workgroups are
// dispatched round-robin over the 8 XCDs, each with its own L2).
__device__ inline unsigned xcd_block(unsigned bid, unsigned nblocks) {
  const unsigned m = nblocks / 8, r = nblocks % 8;
  const unsigned xcd = bid % 8, k = bid / 8;
  return xcd * m + (xcd < r ? xcd : r) + k;
}

constexpr size_t INFINITY_CACHE = (size_t)256 << 20;   // bytes

// Scalar parameters handed to every kernel by value.
struct Geom {
  int nx, ny, nz;
  int periodic_z;
  int dtx, dty, dtz;      // detection tiles per axis (DX x DY x DZ nodes)
  int ltx, lty, ltz;      // lattice blocks per axis (LX x LY x LZ nodes)
  FastDiv fdtx, fdty;     // divisions by dtx, dty
  FastDiv fltx, flty;     // divisions by ltx, lty
  int tile_cap;           // particles per candidate list (both tilings)
  int maxent;             // lattice blocks per particle (partial-sum slots)
  float inv_l[3];         // 1 / period per axis in FP32, 0 on a bounded axis
  int cached;             // both population buffers fit the Infinity Cache
  long long ncell;
};

// Candidate lists of both tilings and the momentum-exchange partial sums.
// dlist[t*cap + s]: particle ids reaching detection tile t.
// llist[b*cap + s]: particle ids reaching lattice block b, lent[b*cap + s]:
// index k of block b in that particle's own block enumeration;
// part[(p*maxent + k)*6 + 0..5] = the (force, torque) the nodes of that
// block contribute to particle p; nent[p] = blocks enumerated for p;
// ovf[p*6 + ..] collects the rare contributions that do not fit the
// per-lane slots.
struct Tiles {
  int* dcount;
  int* dlist;
  int* lcount;
  int* llist;
  int* lent;
  int* nent;
  double* part;
  double* ovf;
  // contact forces of the step, per particle: ccount[p] entries, each with
  // the partner id ckey[p*MAXC + k] (walls -1, -2) and (force, torque)
  // cval[(p*MAXC + k)*6 + 0..5]; summed in partner order by k_particles
  int* ccount;
  int* ckey;
  double* cval;
};

struct Phys {
  double tau, omega;      // relaxation time and 1/tau
  double wall_u[2][3];
  double gravity[3];
  double a_ext[3];        // uniform fluid acceleration (incl. balance 1)
  int bal_mode;           // 2: the acceleration is Counters::bal_a (device)
  double eps, delta_c;
  float eps_h32, eps_q32;  // eps / 2 and 1 / (4 eps) in FP32 (coupling weight)
  int n_c;
  double estar;           // effective modulus, eq. (5)
  double restitution, mu_s, mu_k, u_k;
  double dt_sub;          // length of a contact sub-step (1 / n_sub)
};

// Field read-outs go through pinned chunks of this size, one per worker
// thread, in turn: the device writes one worker's chunk while the others copy
// theirs into the caller's array.
constexpr int READ_WORKERS = 8;
constexpr size_t READ_CHUNK = (size_t)65536 * 36;   // 65536 nodes of density,
                                                    // velocity and owner
constexpr int PART_OUT = 13, FORCE_OUT = 12;        // doubles per particle

constexpr int NKERN = 7;   // clear, treat, particles, keep, detect, lattice, mea

// Device copy of the whole step state (populations f*, particle block,
// candidate lists and partial sums, both pair tables, owner map, counters).
struct Snapshot {
  void* f = nullptr;
  void* part = nullptr;
  void* tiles = nullptr;
  void* psums = nullptr;
  uint64_t* keys[2] = {nullptr, nullptr};
  PairRec* rec[2] = {nullptr, nullptr};
  int* owner = nullptr;
  Counters* ctr = nullptr;
  int cur = 0, tcur = 0;
  long long step = 0;
};

// Recorded forward window of the adjoint and its work arrays.
struct Adjoint {
  bool recorded = false;
  int K = 0, L = 0;                  // steps, steps per checkpoint
  // a block for the snapshots, from the record on, and one for the store and
  // the work arrays, from the first gradient on (or from the record, where its
  // memory is at hand already); each lent (Ctx::adj_mem, Ctx::adj_store) or
  // allocated
  void* block[2] = {nullptr, nullptr};   // those allocated here
  bool store_lent = false;               // the store stands in Ctx::adj_store
  Snapshot* ck = nullptr;            // checkpoint at the start of each segment
  int nseg = 0;
  Snapshot end;                      // state after the K steps
  double* fst = nullptr;             // (L + 1) x Q x ncell: f* at each step of a segment
  int* ost = nullptr;                // (L + 1) x ncell: owner maps
  double* pst = nullptr;             // (L + 1) x np x 22: particle states
  double* frc = nullptr;             // L x np x 12: forces of each step
  int stored = -1;                   // the segment that these four hold
  double* hbar[2] = {nullptr, nullptr};   // dJ/df (Q x ncell), in and out
  double* pbar = nullptr;            // np x 12 particle adjoints
  double* sbar = nullptr;            // np: dJ/ds
  double* work = nullptr;            // adjoint_work_doubles
};

struct Ctx {
  hlbm_params P;
  Geom g;
  Phys ph;
  hipStream_t stream;
  bool own_stream;
  int precision;
  size_t bytes_per_value;
  // populations (two buffers, ping-pong); fbuf[cur] holds f* of the last step
  void* fbuf[2];
  bool own_f;
  int cur;
  // particles
  int np;
  Particles part;         // device pointers
  void* part_block;       // one allocation for all particle arrays
  double* Fh;             // [np][3] hydrodynamic force of the last step
  double* Th;
  double* Fc;             // contact force / torque of the last step
  double* Tc;
  // lattice-side maps
  int* owner;             // [ncell]
  Tiles tl;
  void* tile_block;       // allocation holding count, list, ent
  void* part_sums;        // allocation holding nent, part, ovf
  // contacts
  PairTable tab[2];
  // convex polyhedron types: host records (volume, second moment about the
  // centroid, circumradius at unit scale) and the device table
  struct PolyHost {
    bool ok = false;
    PolyDev dev;
    double vol = 0.0, J[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  } poly_host[MAXPOLY];
  PolyDev* poly_dev = nullptr;
  bool has_poly = false;  // some particle is a polyhedron: kernels with that path
  bool has_ellipsoid = false;  // some particle is an ellipsoid type: the variants
                               // that also evaluate smooth bodies
  int tcur;               // tab[tcur] = current contact list
  Counters* counters;     // device
  double* scratch;        // [ncell] FP64 staging for host conversions
  double* fixed_scratch;  // device address of the fixed staging array
  int device = 0;
  // pinned host memory of the read-outs: the counters and a particle
  // read-out (allocated with the particles), and the chunks of the field
  // read-outs (allocated by the first that needs them), one per worker; each
  // locked by the read-out that uses it
  Counters* host_ctr = nullptr;
  double* host_part = nullptr;
  void* chunk[READ_WORKERS] = {};
  hipEvent_t chunk_ev[READ_WORKERS] = {};
  std::mutex read_mu, chunk_mu;
  double* bal_part = nullptr;  // per-block (mass, momentum) sums, balance mode 2
  // state
  bool particles_ready, fluid_ready;
  long long step;
  // per-kernel timing: ev_per_step events per step, a pool for `tcap` steps
  bool timing;
  int tcap, tused;
  hipEvent_t* tev;
  // sizes of the state blocks (for snapshots)
  size_t part_bytes = 0, tile_bytes = 0, psum_bytes = 0;
  Adjoint adj;
  // device memory lent for the adjoint (hlbm_bind_adjoint,
  // hlbm_bind_adjoint_store), never freed here
  void *adj_mem = nullptr, *adj_store = nullptr;
  size_t adj_mem_bytes = 0, adj_store_bytes = 0;
  // graphs: one per (population parity, contact-table parity) for a single
  // step and one for GRAPH_STEPS steps
  bool use_graph;
  hipGraphExec_t gexec[4];
  bool graph_ready[4];
  hipGraphExec_t gexec_n[4];
  bool graph_n_ready[4] = {};
  bool graph_n_run[4] = {};      // replayed at least once (its one-time
                                 // setup on the device is done)
  int n_sub;
  int ev_per_step;        // timing events per step: 2 + 5 n_sub
  char err[512] = {};     // last error message (fixed: error paths allocate nothing)
};

// ---- launch wrappers (kernels live in the .hip files) --------------------
// Bookkeeping outside the steps (a step leaves everything as the next one
// needs it): CLEAR_TABLE the listed slots of a pair table and the particles'
// contact slots, CLEAR_TILES the detection-tile and lattice-block counts,
// CLEAR_RESULTS the contact forces and the sample counter, CLEAR_ALL_SLOTS
// every slot of the table (once, after allocation); CLEAR_COUNT adds the
// cells of the slots that CLEAR_TABLE empties to the total
constexpr int CLEAR_TABLE = 1, CLEAR_TILES = 2, CLEAR_RESULTS = 4, CLEAR_ALL_SLOTS = 8,
              CLEAR_COUNT = 16;
hipError_t launch_clear(Ctx& c, PairTable table, int what);
// pairs and cells of the detection that filled a table.  The records hold the
// counts already; an atomic per committed tile on shared counters had cost
// detection more than all the rest of it where contacts are many (120^3 nodes,
// 905 settling spheres in contact: 99 us, 14 us without)
hipError_t launch_count(Ctx& c, PairTable table);
// move: 0 bin only, 1 gather the hydrodynamic force and move, 2 move with
// the stored hydrodynamic force (later sub-steps).  bin_blocks: also bin into
// lattice blocks (the last binning before a lattice pass).
// keep_from / keep_to (optional, both or neither): the contact carry-over
// from one pair table to the next, and the clearing of the slots it read,
// run in the same launch; so does (balance) the second stage of the balance
// sums of the last lattice pass
hipError_t launch_particles(Ctx& c, int move, bool bin_blocks,
                            const PairTable* keep_from = nullptr,
                            const PairTable* keep_to = nullptr, bool balance = false);
hipError_t launch_detect(Ctx& c, PairTable to);
// stream-collide src -> dst with the coupling of the current owner map
hipError_t launch_lattice(Ctx& c, const void* src, void* dst);
// momentum exchange over the collided populations fstar (force of the next step)
hipError_t launch_mea(Ctx& c, const void* fstar);
// balance mode 2: the lattice blocks' mass and momentum of f (initial state),
// then the controller (init = 1 at the start, 0 after a collision) from the
// block sums
hipError_t launch_pop_moments(Ctx& c, const void* f);
hipError_t launch_balance(Ctx& c, int init);
// treatment of table t; next: the table that the carry-over and detection will
// fill (its slots are clear already; its list count is reset here); balance:
// the first stage of the balance sums in the same launch
hipError_t launch_treat(Ctx& c, PairTable t, PairTable next, bool balance);
hipError_t launch_fill_equilibrium(Ctx& c, void* f, double rho,
                                   const double u[3]);
hipError_t launch_store_direction(Ctx& c, void* f, int i, const double* src);
// Read-outs of the nodes (populations: values) begin .. begin + count into
// host or device memory; null pointers skip.
// populations f* as FP64, all directions one after another
hipError_t launch_load_populations(Ctx& c, const void* f, long long begin, long long count,
                                   double* dst);
// density, velocity (three per node) and owner
hipError_t launch_moments(Ctx& c, const void* f, long long begin, long long count, double* rho,
                          double* u, int* owner);
// coupling weight and particle velocity (three per node)
hipError_t launch_coupling_field(Ctx& c, long long begin, long long count, double* B, double* up);
// n doubles and the counters
hipError_t launch_export(Ctx& c, const double* src, long long n, double* dst, Counters* dst_ctr);
// nodes the fixed staging array of hlbm_read_coupling_noalloc holds
constexpr long long NOALLOC_MAX_CELLS = 1LL << 21;
hipError_t noalloc_scratch(double** out);
// adjoint (k_adjoint.hip)
int adjoint_record_doubles();
int adjoint_slots();
size_t adjoint_work_doubles(const Ctx& c);
// particle records and (frc given) the forces of the last step
hipError_t launch_record(Ctx& c, double* prec, double* frc);
hipError_t launch_fill_zero(Ctx& c, double* p, long long n);
// reverse of the motion of a step: prec its particle records, frc its forces
hipError_t launch_adjoint_move(Ctx& c, const double* prec, const double* frc, double* pbar,
                               double* sbar, double* work);
// reverse of the momentum exchange of the next step and of the collision of
// this one (hin: dJ/df of the next step; hout null, the initial state: no
// collision; fown: f* of this step, fprev: of the one before)
hipError_t launch_adjoint_node(Ctx& c, double* hin, double* hout, const double* fown,
                               const double* fprev, const int* owner, const double* prec,
                               double* pbar, double* work);

}  // namespace hlbm
