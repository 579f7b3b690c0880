// Velocity Verlet in FP64 (Section 2, Fig. 3 box 5):
//   kick  v += dt/(2m) F,   drift  x <- wrap(x + dt v),   kick again after F.
#include "dcm_device.hpp"
#include "dcm_internal.hpp"

namespace dcm {

// A workgroup's share of sum_i v_i^2 (the threads' acc), in a fixed order.
__device__ __forceinline__ void kinetic_partial(double acc, double *partials) {
  __shared__ double red[4];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// KE: also the workgroups' sums of v^2 after the kick
template <bool KE>
__global__ __launch_bounds__(256) void k_kick(double *__restrict__ vx, double *__restrict__ vy,
                                              double *__restrict__ vz,
                                              const double *__restrict__ fx,
                                              const double *__restrict__ fy,
                                              const double *__restrict__ fz, int64_t n,
                                              double c, double *ke) {
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double a = vx[i] + c * fx[i], b = vy[i] + c * fy[i], d = vz[i] + c * fz[i];
    vx[i] = a;
    vy[i] = b;
    vz[i] = d;
    if constexpr (KE) acc += (a * a + b * b) + d * d;
  }
  if constexpr (KE) kinetic_partial(acc, ke);
}

__global__ __launch_bounds__(256) void k_kick_drift(
    double *__restrict__ x, double *__restrict__ y, double *__restrict__ z,
    double *__restrict__ vx, double *__restrict__ vy, double *__restrict__ vz,
    const double *__restrict__ fx, const double *__restrict__ fy, const double *__restrict__ fz,
    int64_t n, double c, double dt, double Lx, double Ly, double Lz) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double a = vx[i] + c * fx[i];
    double b = vy[i] + c * fy[i];
    double d = vz[i] + c * fz[i];
    vx[i] = a;
    vy[i] = b;
    vz[i] = d;
    x[i] = wrap_coord(x[i] + dt * a, Lx);
    y[i] = wrap_coord(y[i] + dt * b, Ly);
    z[i] = wrap_coord(z[i] + dt * d, Lz);
  }
}

// The closing kick of one step and the opening kick and drift of the next
// in one pass over the particles: the same operations in the same order as
// k_kick followed by k_kick_drift, without the round trip of v through HBM.
// KE: also the workgroups' sums of v^2 between the kicks (an energy series is
// recorded; the kick, the sums and the next drift were three passes).
// BIN: also the density binning of the next step's detection (Section
// 2.1) from the new positions while they are in registers: counts[v] += 1
// for the voxel v of each particle, as the binning pass computes it (the
// positions written here are wrapped already, and wrapping them again gives
// them back unchanged).  A non-finite position is flagged and not binned.
// Uniform trip count: every lane of a wavefront reaches the aggregated add.
struct DensityBins {
  int nx, ny, nz;
  double sx, sy, sz;
  uint32_t *counts, *status;
};
template <bool KE, bool BIN>
__global__ __launch_bounds__(256) void k_kick_kick_drift(
    double *__restrict__ x, double *__restrict__ y, double *__restrict__ z,
    double *__restrict__ vx, double *__restrict__ vy, double *__restrict__ vz,
    const double *__restrict__ fx, const double *__restrict__ fy, const double *__restrict__ fz,
    int64_t n, double c, double dt, double Lx, double Ly, double Lz, double *ke, DensityBins bins) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double acc = 0.0;
  for (int64_t base = blockIdx.x * (int64_t)blockDim.x; base < n; base += stride) {
    const int64_t i = base + threadIdx.x;
    bool valid = i < n;
    uint32_t vox = 0;
    if (valid) {
      const double gx = c * fx[i], gy = c * fy[i], gz = c * fz[i];
      const double ex = vx[i] + gx, ey = vy[i] + gy, ez = vz[i] + gz;
      if constexpr (KE) acc += (ex * ex + ey * ey) + ez * ez;
      const double a = ex + gx;
      const double b = ey + gy;
      const double d = ez + gz;
      vx[i] = a;
      vy[i] = b;
      vz[i] = d;
      const double px = wrap_coord(x[i] + dt * a, Lx);
      const double py = wrap_coord(y[i] + dt * b, Ly);
      const double pz = wrap_coord(z[i] + dt * d, Lz);
      x[i] = px;
      y[i] = py;
      z[i] = pz;
      if constexpr (BIN) {
        if (!finite3(px, py, pz)) {
          atomicOr(bins.status, ST_NONFINITE_POS);
          valid = false;
        } else {
          const int cx = slab_index(wrap_coord(px, Lx), bins.sx, bins.nx);
          const int cy = slab_index(wrap_coord(py, Ly), bins.sy, bins.ny);
          const int cz = slab_index(wrap_coord(pz, Lz), bins.sz, bins.nz);
          vox = (uint32_t)(((int64_t)cz * bins.ny + cy) * bins.nx + cx);
        }
      }
    }
    if constexpr (BIN) wave_run_add(bins.counts, vox, valid);
  }
  if constexpr (KE) kinetic_partial(acc, ke);
}

static unsigned grid_for(int64_t n) {
  int64_t b = ceil_div(n, 256);
  if (b < 1) b = 1;
  if (b > 16384) b = 16384;
  return (unsigned)b;
}

// Kinetic energy sum_i m v_i^2 / 2: fixed-size grid of block partials, then
// one workgroup sums them in a fixed order.
constexpr int kKeBlocks = 1024;
int64_t kinetic_blocks(int64_t n) {
  (void)n;
  return kKeBlocks;
}

void launch_kick(hipStream_t s, double *vx, double *vy, double *vz, const double *fx,
                 const double *fy, const double *fz, int64_t n, double c, double *ke) {
  if (ke)
    hipLaunchKernelGGL(k_kick<true>, dim3(kKeBlocks), dim3(256), 0, s, vx, vy, vz, fx, fy, fz, n,
                       c, ke);
  else if (n > 0)
    hipLaunchKernelGGL(k_kick<false>, dim3(grid_for(n)), dim3(256), 0, s, vx, vy, vz, fx, fy, fz,
                       n, c, nullptr);
}

void launch_kick_drift(hipStream_t s, double *x, double *y, double *z, double *vx, double *vy,
                       double *vz, const double *fx, const double *fy, const double *fz,
                       int64_t n, double c, double dt, const double L[3]) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_kick_drift, dim3(grid_for(n)), dim3(256), 0, s, x, y, z, vx, vy, vz, fx,
                     fy, fz, n, c, dt, L[0], L[1], L[2]);
}

void launch_kick_kick_drift(hipStream_t s, double *x, double *y, double *z, double *vx,
                            double *vy, double *vz, const double *fx, const double *fy,
                            const double *fz, int64_t n, double c, double dt, const double L[3],
                            double *ke, const int32_t *nv, const double *sc, uint32_t *counts,
                            uint32_t *status) {
  if (n <= 0 && !ke) return;
  DensityBins b = {};
  if (counts) b = {nv[0], nv[1], nv[2], sc[0], sc[1], sc[2], counts, status};
  const dim3 g(ke ? (unsigned)kKeBlocks : grid_for(n)), t(256);
#define LAUNCH(KE, BIN)                                                                        \
  hipLaunchKernelGGL((k_kick_kick_drift<KE, BIN>), g, t, 0, s, x, y, z, vx, vy, vz, fx, fy, fz, \
                     n, c, dt, L[0], L[1], L[2], ke, b)
  if (ke && counts) LAUNCH(true, true);
  else if (ke) LAUNCH(true, false);
  else if (counts) LAUNCH(false, true);
  else LAUNCH(false, false);
#undef LAUNCH
}

// A step's two energies, a workgroup each: the pair energy from the force
// pass's partials (rows of kPartialSlots, slot 0), summed as the force entry
// points sum it, and the kinetic energy from the kick's.
__global__ __launch_bounds__(kReduceThreads) void k_step_energies(
    const double *__restrict__ pair, int64_t rows, const double *__restrict__ ke, double half_m,
    double *out) {
  __shared__ double red[kReduceThreads / 64][1];
  if (blockIdx.x == 0) {
    double t[1];
    sum_rows<kReduceThreads, 1, kPartialSlots>(pair, rows, red, t);
    if (threadIdx.x == 0) out[0] = t[0];
    return;
  }
  double acc = 0.0;
  if (threadIdx.x < 256)
    for (int64_t b = threadIdx.x; b < kKeBlocks; b += 256) acc += ke[b];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[1] = half_m * (((red[0][0] + red[1][0]) + red[2][0]) + red[3][0]);
}

void launch_step_energies(hipStream_t s, const double *pair, int64_t rows, const double *ke,
                          double mass, double *out) {
  hipLaunchKernelGGL(k_step_energies, dim3(2), dim3(kReduceThreads), 0, s, pair, rows, ke,
                     0.5 * mass, out);
}

}  // namespace dcm
