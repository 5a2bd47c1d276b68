// Read-out kernels: the coupling field (Sec. 3.2), the particle state and the
// counters; and the fixed device staging array of the read-out that allocates
// nothing.
#include <mutex>

#include "context.h"

namespace hlbm {

namespace {

// Staging of hlbm_read_coupling_noalloc: B for every node, then u_p
// interleaved per node (4 doubles per node, NOALLOC_MAX_CELLS nodes at most,
// 64 MiB).  Each device holds its own copy for the life of the process; in
// host code the name only stands for the symbol, and kernels get the
// device address that hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) double scratch[4 * (size_t)NOALLOC_MAX_CELLS];

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[MAX_DEVICES] = {};

// Coupling field at the current particle state (Sec. 3.2), FP64, of the nodes
// begin .. begin + count: the weight B(d_owner) to B (may be null) and u_p =
// U + w x r of the owner, three per node, to up (may be null); 0 where no
// particle owns the node.
__global__ __launch_bounds__(256) void k_coupling_field(const int* __restrict__ owner,
                                                        Particles P, Geom g, Phys ph,
                                                        long long begin, long long count,
                                                        double* __restrict__ B,
                                                        double* __restrict__ up) {
  __shared__ double sh[3 * 256];
  const long long at = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long id = begin + at;
  const int o = at < count ? owner_id(owner[id]) : -1;
  double b = 0.0, v[3] = {0.0, 0.0, 0.0};
  if (o >= 0) {
    const int x = (int)(id % g.nx), y = (int)((id / g.nx) % g.ny);
    const int z = (int)(id / ((long long)g.nx * g.ny));
    const double r[3] = {minimg((double)x - P.X[3 * o], (double)g.nx, true),
                         minimg((double)y - P.X[3 * o + 1], (double)g.ny, true),
                         minimg((double)z - P.X[3 * o + 2], (double)g.nz, g.periodic_z != 0)};
    if (B)
      b = weight(sdf<true>(P.shape[o], P.size[o], P.R + 9 * o, r[0], r[1], r[2], P.poly), ph.eps);
    const double* W = P.W + 3 * o;
    v[0] = P.U[3 * o] + (W[1] * r[2] - W[2] * r[1]);
    v[1] = P.U[3 * o + 1] + (W[2] * r[0] - W[0] * r[2]);
    v[2] = P.U[3 * o + 2] + (W[0] * r[1] - W[1] * r[0]);
  }
  if (B && at < count) B[at] = b;
  if (up) store_rows3(sh, v, (long long)blockIdx.x * 256, count, up);
}

// n doubles and the counters to host memory.
__global__ __launch_bounds__(256) void k_export(const double* __restrict__ src, long long n,
                                                const Counters* __restrict__ ctr,
                                                double* __restrict__ dst,
                                                Counters* __restrict__ dst_ctr) {
  const long long stride = (long long)gridDim.x * 256;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += stride)
    dst[i] = src[i];
  const unsigned words = sizeof(Counters) / sizeof(unsigned long long);
  if (blockIdx.x == 0 && threadIdx.x < words)
    ((unsigned long long*)dst_ctr)[threadIdx.x] =
        ((const unsigned long long*)ctr)[threadIdx.x];
}
static_assert(sizeof(Counters) % sizeof(unsigned long long) == 0, "counters copied by words");

}  // namespace

hipError_t launch_coupling_field(Ctx& c, long long begin, long long count, double* B, double* up) {
  hipLaunchKernelGGL(k_coupling_field, dim3((unsigned)((count + 255) / 256)), dim3(256), 0,
                     c.stream, c.owner, c.part, c.g, c.ph, begin, count, B, up);
  return hipGetLastError();
}

hipError_t launch_export(Ctx& c, const double* src, long long n, double* dst, Counters* dst_ctr) {
  const long long blocks = (n + 1023) / 1024;
  hipLaunchKernelGGL(k_export, dim3((unsigned)(blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks))),
                     dim3(256), 0, c.stream, src, n, c.counters, dst, dst_ctr);
  return hipGetLastError();
}

// Device address of the staging array on the current device, looked up once
// per device (first context created there) and kept.
hipError_t noalloc_scratch(double** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    double* ptr = nullptr;
    e = hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace hlbm
