// Cutoff-limited fast-sweeping distances (Section 2.2, Algorithm 2.1).
//
// Every voxel applies the first-order Godunov upwind update of |grad d| = 1,
// d <- min(d, G(neighbours)), accepting only values <= rc_grid, until nothing
// changes.  The update is monotone, so any order of updates reaches the same
// fixed point as the paper's sweeps; source voxels (interface and
// low-density phase) hold 0 and are never rewritten.
//
// Tiles use temporal blocking: a launch stages a tile and a frozen one-voxel
// halo in LDS, iterates synchronous sub-waves inside, and writes the tile.
// Like the paper's queue of boxes next to updated boxes, a tile only runs
// again when it changed in the previous launch, or a voxel next to one of its
// faces did; a launch in which no tile changes ends the sweep.  Launches read
// one global buffer and write the other, so the result does not depend on
// scheduling.  Thin grids of dcm_sweep_distance, whose caller counts the
// waves, use plain synchronous waves over all voxels.
#include "dcm_device.hpp"
#include "dcm_internal.hpp"

namespace dcm {

constexpr int TX = 16, TY = 8, TZ = 8;                // tile
constexpr int QX = TX + 2, QY = TY + 2, QZ = TZ + 2;  // with halo
// LDS pitches of a row and a plane (doubles): the half wavefront that reads two
// planes of a 4 x 4 x 4 block meets 64 different banks (without the padding
// half of them twice: 2 to 3% of a pass)
constexpr int PX = QX + 2, PXY = QY * PX + 8;
static_assert(2 * PX % 64 == 40 && 2 * PXY % 64 == 32, "bank spread of a block");
constexpr int kTileThreads = TX * TY * TZ;            // one voxel per thread
constexpr int kTileWaves = kTileThreads / 64;

bool fsm_tiled(const int32_t nv[3]) {
  return nv[0] >= TX + 2 && nv[1] >= TY + 2 && nv[2] >= TZ + 2;
}

int64_t fsm_tile_count(const int32_t nv[3]) {
  return ceil_div(nv[0], TX) * ceil_div(nv[1], TY) * ceil_div(nv[2], TZ);
}

// Initial distances and the first pass's tile flags, a workgroup to a region
// of kInitX x TY x TZ voxels (kInitX / TX tiles): sources (low-density phase
// and interface) start at 0, the rest at +inf.  A tile holding a source is
// flagged as changed before the first pass: only next to a source can a pass
// change anything at first.  (Where the interface is that of the phase map, a
// tile with a voxel that is not a source then runs at first if it or a face
// neighbour holds an interface voxel; a caller's maps may be others.)  Also
// clears the pass flags and the tiles' stamps, which took a launch of their own
// before.  Bound by the two fields it writes (39 us on the 160 x 160 x 400 grid,
// 4.2 TB/s; 50 to 60 us beside the cell build).
constexpr int kInitX = 64;
struct FsmInit {
  int nx, ny, nz, ntx, nty;
  int nbx;  // regions along x (nty along y)
  double *dA, *dB;
  uint8_t *first;   // tiles holding a source; null: no tiles
  uint8_t *live;    // tiles with a voxel that is not a source
  uint32_t *stamp, *changed;  // cleared
  uint32_t *flags;  // pass flags and list counts, cleared
  int nflags;
};

// A workgroup's region.  The grid is one-dimensional: its other dimensions end at
// 65,535 workgroups, which a long thin grid of voxels passes.
struct InitRegion {
  int x, y, z;
};
__device__ __forceinline__ InitRegion init_region(const FsmInit &p) {
  const int b = (int)blockIdx.x, r = b / p.nbx;
  return {b - r * p.nbx, r % p.nty, r / p.nty};
}

// source(x, y, z): whether the voxel is a source.  prepare: called by the whole
// workgroup first.
template <typename P, typename F>
__device__ __forceinline__ void fsm_init_region(const FsmInit &p, P &&prepare, F &&source) {
  __shared__ int has[kInitX / TX], lives[kInitX / TX];
  const int lx = threadIdx.x & (kInitX - 1), row = threadIdx.x / kInitX;
  const InitRegion at = init_region(p);
  const int x = at.x * kInitX + lx, y0 = at.y * TY, z0 = at.z * TZ;
  if (threadIdx.x < kInitX / TX) has[threadIdx.x] = lives[threadIdx.x] = 0;
  for (int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x; f < p.nflags;
       f += 256 * (int64_t)gridDim.x)
    p.flags[f] = 0u;
  prepare();
  __syncthreads();
  bool any = false, inf = false;
  if (x < p.nx)
#pragma unroll 4
    for (int r = row; r < TY * TZ; r += 256 / kInitX) {
      const int y = y0 + r % TY, z = z0 + r / TY;
      if (y >= p.ny || z >= p.nz) continue;
      const double d = source(x, y, z) ? 0.0 : __builtin_huge_val();
      const int64_t v = ((int64_t)z * p.ny + y) * p.nx + x;
      p.dA[v] = d;
      p.dB[v] = d;
      any |= d == 0.0;
      inf |= d != 0.0;
    }
  if (any) has[lx / TX] = 1;
  if (inf) lives[lx / TX] = 1;
  __syncthreads();
  const int tx = at.x * (kInitX / TX) + threadIdx.x;
  if (p.first && threadIdx.x < kInitX / TX && tx < p.ntx) {
    const int64_t t = ((int64_t)at.z * p.nty + at.y) * p.ntx + tx;
    p.first[t] = (uint8_t)has[threadIdx.x];
    p.live[t] = (uint8_t)lives[threadIdx.x];
    p.stamp[t] = p.changed[t] = 0u;
  }
}

__global__ __launch_bounds__(256) void k_fsm_init(const uint8_t *__restrict__ seg,
                                                  const uint8_t *__restrict__ iface, FsmInit p) {
  fsm_init_region(p, [] {}, [&](int x, int y, int z) {
    const int64_t v = ((int64_t)z * p.ny + y) * p.nx + x;
    return seg[v] == 0 || iface[v] != 0;
  });
}

// The same from the bit-packed phase maps of the regularisation passes
// (final_phase_map), without the byte maps: a voxel starts at +inf iff it
// and its six face neighbours (periodic) are all high density -- otherwise
// it is low density or an interface voxel, a source.  Four threads per row of
// the region form the mask of its 64 voxels, from whole words, in LDS: a look
// at seven bits per voxel was a chain of loads per row, and the workgroups of a
// small grid took 13 us for it.
__global__ __launch_bounds__(256) void k_fsm_init_bits(const uint32_t *b0, const uint32_t *b1,
                                                       const Ctl *ctl, FsmInit p) {
  __shared__ unsigned long long inner[TY * TZ], parts[4][TY * TZ];
  static_assert(kInitX == 64 && TY * TZ == 64, "two words a row, 64 rows, 4 threads a row");
  const int nx = p.nx, ny = p.ny, nz = p.nz, W = (nx + 31) >> 5;
  fsm_init_region(
      p,
      [&] {
        const int r = threadIdx.x & 63, part = threadIdx.x >> 6;
        const InitRegion at = init_region(p);
        const int y = at.y * TY + r % TY, z = at.z * TZ + r / TY;
        if (y < ny && z < nz) {
          const uint32_t *__restrict__ s =
              final_phase_map(ctl->maj_chg1, ctl->maj_chg2, kMajorityMaxPasses, b0, b1);
          const int k = at.x * 2;
          auto row = [&](int yy, int zz) {
            const uint32_t *q = s + ((int64_t)zz * ny + yy) * W + k;
            return (unsigned long long)q[0] | (k + 1 < W ? (unsigned long long)q[1] << 32 : 0ull);
          };
          unsigned long long a;
          if (part == 0) {
            const uint32_t *own = s + ((int64_t)z * ny + y) * W;
            const unsigned long long m = row(y, z);
            // bits x - 1 and x + 1 at the place of x
            const unsigned long long before =
                k == 0 ? own[W - 1] >> ((nx - 1) & 31) & 1u : own[k - 1] >> 31;
            unsigned long long after = m >> 1;
            const int last = nx - 1 - k * 32;  // place of the row's last voxel
            if (last < 64) after |= (unsigned long long)(own[0] & 1u) << last;
            else after |= (unsigned long long)(own[k + 2] & 1u) << 63;
            a = m & (m << 1 | before) & after;
          } else if (part == 1) {
            a = row(y == 0 ? ny - 1 : y - 1, z) & row(y + 1 == ny ? 0 : y + 1, z);
          } else {
            a = row(y, part == 2 ? (z == 0 ? nz - 1 : z - 1) : (z + 1 == nz ? 0 : z + 1));
          }
          parts[part][r] = a;
        }
        __syncthreads();
        if (part == 0) inner[r] = parts[0][r] & parts[1][r] & parts[2][r] & parts[3][r];
      },
      [&](int x, int y, int z) {
        return !(inner[(z % TZ) * TY + y % TY] >> (x & (kInitX - 1)) & 1ull);
      });
}

// Godunov solve: with the smaller face neighbour a_k and spacing h_k per axis
// (w_k = 1/h_k^2), d solves sum over the m smallest a_k of w_k (d - a_k)^2 = 1
// for the largest m whose root does not pass the next a_k; written relative
// to the smallest a.
//
// The sums of the w over the two smallest (all) axes depend only on the axis
// left out (added last), so they and their reciprocals are uniform values
// (SweepGeom) indexed by the axis of the largest a.  A quotient x / A is then
// q = x r with r = 1/A correctly rounded, corrected once by its exact
// remainder, which gives the correctly rounded quotient (P. Markstein, IBM J.
// Res. Dev. 34, 1990).  For the square root see root_of.
struct SweepGeom {
  int nx, ny, nz;
  double h[3], w[3];
  double a2[3], r2[3];  // w_i + w_j of the two axes other than k, and its reciprocal
  double a3[3], r3[3];  // (w_i + w_j) + w_k, and its reciprocal
  double rc_grid;
};

__device__ __forceinline__ double by_axis(const double v[3], int k) {
  return k == 0 ? v[0] : (k == 1 ? v[1] : v[2]);
}

__device__ __forceinline__ double div_by(double x, double A, double r) {
  const double q = x * r;
  return fma(fma(-q, A, x), r, q);
}

// Square root of v, 0 or of the size that spacings between 1e-130 and 1e130 give
// (w rounded off at its last place, to ten w).  With y near 1 / sqrt(v) from the
// hardware and e = 1 - v y^2, the binomial series of (1 - e)^(-1/2) gives
// 1 / sqrt(v) = y (1 + e / 2 + 3 e^2 / 8 + ...): one step of third order (A. S.
// Householder, The Numerical Treatment of a Single Nonlinear Equation, 1970),
// which leaves 5 e^3 / 16, below a rounding for e under 2^-18.  g = v y1 is then
// within three units of its last place of the root, and g + r y1 / 2, r its
// remainder v - g^2 (Markstein, as above), within a few 2^-52 of a unit before
// its one rounding.  (3 to 5% of a sweep against the library's, which must serve
// every argument: 10 million voxels, interface everywhere, 4478 and 4308 us.)
__device__ __forceinline__ double root_of(double v) {
  const double y = __builtin_amdgcn_rsq(v);
  const double e = fma(-(v * y), y, 1.0);
  const double y1 = fma(y * e, fma(0.375, e, 0.5), y);
  const double g = v * y1;
  const double s = fma(fma(-g, g, v), 0.5 * y1, g);
  return v == 0.0 ? 0.0 : s;
}

// ISO: equal spacings on every axis, so only the a's need ordering
template <bool ISO>
__device__ __forceinline__ double godunov(double a0, double a1, double a2, const SweepGeom &g) {
  int k0 = 0, k1 = 1, k2 = 2;
  // ascending, keeping axis order on ties
  auto order = [](double &p, double &q, int &kp, int &kq) {
    const bool s = q < p;
    const double t = s ? q : p;
    q = s ? p : q;
    p = t;
    if constexpr (!ISO) {
      const int kt = s ? kq : kp;
      kq = s ? kp : kq;
      kp = kt;
    }
  };
  order(a0, a1, k0, k1);
  order(a1, a2, k1, k2);
  order(a0, a1, k0, k1);
  const double h0 = ISO ? g.h[0] : by_axis(g.h, k0);
  const double w1 = ISO ? g.w[0] : by_axis(g.w, k1), w2 = ISO ? g.w[0] : by_axis(g.w, k2);
  const double A2 = ISO ? g.a2[0] : by_axis(g.a2, k2), R2 = ISO ? g.r2[0] : by_axis(g.r2, k2);
  const double A3 = ISO ? g.a3[0] : by_axis(g.a3, k2), R3 = ISO ? g.r3[0] : by_axis(g.r3, k2);
  const double b1 = a1 - a0, b2 = a2 - a0;
  const double d1 = a0 + h0;
  // a root that no lane of the wavefront needs is not formed (a flat front
  // along an axis needs neither); an infinite a makes the roots it enters NaN,
  // and they are not chosen
  double d = d1;
  bool more = !(d1 <= a1);
  if (__ballot(more) != 0ull) {
    const double p1 = w1 * b1, p2 = w2 * b2;
    double disc2 = p1 * p1 - A2 * (p1 * b1 - 1.0);
    disc2 = disc2 < 0.0 ? 0.0 : disc2;
    const double d2 = a0 + div_by(p1 + root_of(disc2), A2, R2);
    d = more ? d2 : d;
    more = more && !(d2 <= a2);
    if (__ballot(more) != 0ull) {
      const double B3 = p1 + p2;
      double disc3 = B3 * B3 - A3 * ((p1 * b1 + p2 * b2) - 1.0);
      disc3 = disc3 < 0.0 ? 0.0 : disc3;
      const double d3 = a0 + div_by(B3 + root_of(disc3), A3, R3);
      d = more ? d3 : d;
    }
  }
  return isinf(a0) ? a0 : d;
}

// ------------------------------------------------------------- tiled sweep
// Launch L reads buf[(L-1)&1] and writes buf[L&1] for its active tiles.
// Active in the first launch are the tiles with a source and their face
// neighbours (found from the init's flags, or listed by k_fsm_first); a
// tile that changes in launch L puts itself, and the face neighbours next to a
// voxel that changed, on launch L + 1's list (stamp: the last launch a tile was
// listed for).  live: tiles with a voxel that is not a source; the others never
// run.
//
// With last > launch the launch goes on with the passes up to `last` (TAIL).
// Its workgroups take the tiles of a pass from the list one by one, and wait at
// the pass's end until as many are finished as were listed.  A workgroup waits
// only when no tile is left to take, so each of those it waits for is in the
// hands of one that is running: the wait ends whether or not the others have
// started, and one that starts late finds nothing to take and catches up.
//
// A pass is bound by latency: one after the other, the sub-waves of the tiles
// that the front crosses, each a solve (97 vector instructions, 69 of them
// FP64, where all three axes count) and a barrier long.  So one thread owns
// one voxel, in a register; a wavefront owns a 4 x 4 x 4 block, so that a
// front of any direction touches few blocks; one bit per block says that a
// sub-wave changed it, and the next sub-wave solves only the blocks that
// changed or have a face neighbour that did; two copies of the tile in LDS,
// written in turn, leave one barrier to a sub-wave; and the lists spread the
// active tiles evenly over the workgroups.
// Sweep of a step, all passes, before (256 threads solving a 16 x 8 x 8 tile's
// 1024 voxels in every sub-wave, the active tiles found by a look at all 26
// neighbours of every tile) and after: 120^3 grid, droplet 326 -> 160 us;
// 200 x 100 x 100, cylinder 419 -> 285 us; 160 x 160 x 400 settled (64 passes
// launched, then 15) 354 -> 225 us.
struct SweepTiles {
  int ntx, nty, ntz;
  const uint8_t *first, *live;
  uint32_t *stamp, *changed;  // last launch listed for; last launch that changed the tile
  uint32_t *count;            // [launch]: entries of the launch's list
  uint32_t *taken, *done;     // [launch]: entries taken and finished (TAIL)
  int32_t *list[2];           // of even and odd launches
};

__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// face neighbour k (0 .. 5: -x +x -y +y -z +z) of the tile (tx, ty, tz),
// periodic; 6: the tile itself
__device__ __forceinline__ int near_tile(const SweepTiles &w, int tx, int ty, int tz, int k) {
  int x = tx + (k == 1) - (k == 0), y = ty + (k == 3) - (k == 2), z = tz + (k == 5) - (k == 4);
  x = x < 0 ? w.ntx - 1 : (x == w.ntx ? 0 : x);
  y = y < 0 ? w.nty - 1 : (y == w.nty ? 0 : y);
  z = z < 0 ? w.ntz - 1 : (z == w.ntz ? 0 : z);
  return (z * w.nty + y) * w.ntx + x;
}

// The first launch's list on a grid of more tiles than workgroups: without it
// each workgroup looks through its share of the tiles, and the few whose share
// holds two or three active ones set the time.
__global__ __launch_bounds__(256) void k_fsm_first(SweepTiles w) {
  const int ntiles = w.ntx * w.nty * w.ntz, t = (int)(blockIdx.x * 256 + threadIdx.x);
  bool act = false;
  if (t < ntiles) {
    const int tx = t % w.ntx, tr = t / w.ntx, ty = tr % w.nty, tz = tr / w.nty;
    int seen = 0;
#pragma unroll
    for (int k = 0; k < 7; ++k) seen |= w.first[near_tile(w, tx, ty, tz, k)];
    act = seen != 0 && w.live[t] != 0;
  }
  const unsigned long long m = __ballot(act);
  const int lane = threadIdx.x & 63;
  uint32_t base = 0;
  if (lane == 0 && m) base = atomicAdd(&w.count[1], (uint32_t)__popcll(m));
  base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
  if (act) w.list[1][base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = t;
}

// Looks at a pass's count of finished tiles, some 0.5 us apart, before a waiting
// workgroup gives up (seconds; a pass takes microseconds): the sweep is then
// reported as not converged instead of hanging.
constexpr unsigned kTailSpins = 1u << 23;

__device__ __forceinline__ uint32_t agent_load(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool ISO, bool TAIL>
__global__ __launch_bounds__(kTileThreads) void k_fsm_tiles(double *dA, double *dB, SweepTiles w,
                                                            SweepGeom g, int launch, int last,
                                                            bool listed, int max_sub,
                                                            uint32_t *flags) {
  constexpr int NT = kTileThreads, BX = TX / 4;
  static_assert(TY == 8 && TZ == 8, "two blocks of 4 along y and z");
  __shared__ double A[2][QZ * PXY];
  __shared__ unsigned int map[3];  // blocks changed by sub-waves 0, 1, 2 mod 3
  __shared__ unsigned int faces;   // the tile's faces (as near_tile) with a changed voxel
  __shared__ unsigned long long todo_s[kTileWaves];  // first launch: active tiles, 64 a wavefront
  __shared__ int got, gave_up;  // TAIL: the entry taken; the wait was given up
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ntiles = w.ntx * w.nty * w.ntz;
  // this thread's voxel in the tile, and its place in LDS
  const int bx = wave % BX, by = (wave / BX) & 1, bz = wave / (2 * BX);
  const int lx = bx * 4 + (lane & 3), ly = by * 4 + ((lane >> 2) & 3), lz = bz * 4 + (lane >> 4);
  const int at = (lz + 1) * PXY + (ly + 1) * PX + lx + 1;
  // this wavefront's block and its face neighbours
  const unsigned int near = (1u << wave) | (bx > 0 ? 1u << (wave - 1) : 0u) |
                            (bx + 1 < BX ? 1u << (wave + 1) : 0u) |
                            (1u << (by ? wave - BX : wave + BX)) |
                            (1u << (bz ? wave - 2 * BX : wave + 2 * BX));
  for (; launch <= last; ++launch) {
    const double *src = (launch & 1) ? dA : dB;
    double *dst = (launch & 1) ? dB : dA;
    // a pass runs only while the previous one changed something
    int entries = 0;
    const bool from_list = TAIL || launch > 1 || listed;
    if (from_list) {
      entries = (int)agent_load(&w.count[launch]);
      if (entries == 0) return;
    }
    bool any_changed = false;
    // this workgroup's share of the list; in the first launch, of all tiles
    // (blockIdx.x, + gridDim.x, ...), looked through NT at a time
    int64_t at_entry = blockIdx.x, t0 = (int64_t)blockIdx.x - NT * (int64_t)gridDim.x;
    int group = 0, groups = 0;
    unsigned long long todo = 0ull;
    while (true) {
      int t;
      if (from_list) {
        if constexpr (TAIL) {
          if (tid == 0) got = (int)atomicAdd(&w.taken[launch], 1u);
          __syncthreads();
          at_entry = __builtin_amdgcn_readfirstlane(got);
        }
        if (at_entry >= entries) break;
        t = __builtin_amdgcn_readfirstlane(
            (int)agent_load((const uint32_t *)&w.list[launch & 1][at_entry]));
        at_entry += gridDim.x;
      } else {
        while (todo == 0ull && group + 1 < groups) todo = uniform_u64(todo_s[++group]);
        if (todo == 0ull) {
          t0 += NT * (int64_t)gridDim.x;
          if (t0 >= ntiles) break;
          __syncthreads();  // todo_s has been read
          const int64_t tl = t0 + (int64_t)tid * gridDim.x;
          bool act = false;
          if (tl < ntiles) {
            const int alive = w.live[tl];
            const int tx = (int)tl % w.ntx, tr = (int)tl / w.ntx, ty = tr % w.nty, tz = tr / w.nty;
            int seen = 0;
#pragma unroll
            for (int k = 0; k < 7; ++k) seen |= w.first[near_tile(w, tx, ty, tz, k)];
            act = seen != 0 && alive != 0;
          }
          const unsigned long long m = __ballot(act);
          if (lane == 0) todo_s[wave] = m;
          __syncthreads();
          group = 0;
          groups = kTileWaves;
          todo = uniform_u64(todo_s[0]);
          continue;
        }
        const int bit = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        t = (int)(t0 + (64 * group + bit) * (int64_t)gridDim.x);
      }
      const int tx = t % w.ntx, tr = t / w.ntx, ty = tr % w.nty, tz = tr / w.nty;
      const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
      const bool owned = x0 + lx < g.nx && y0 + ly < g.ny && z0 + lz < g.nz;
      const bool prev = launch > 1 && agent_load(&w.changed[t]) == (uint32_t)(launch - 1);
      // stage the tile and its halo (periodic; on a grid thinner than the
      // tile a halo voxel copies one of the tile, frozen as any halo voxel)
      for (int e = tid; e < QZ * QY * QX; e += NT) {
        const int ez = e / (QY * QX), r = e - ez * (QY * QX), ey = r / QX, ex = r - ey * QX;
        int gx = x0 + ex - 1, gy = y0 + ey - 1, gz = z0 + ez - 1;
        gx = gx < 0 ? gx + g.nx : (gx >= g.nx ? gx - g.nx : gx);
        gy = gy < 0 ? gy + g.ny : (gy >= g.ny ? gy - g.ny : gy);
        gz = gz < 0 ? gz + g.nz : (gz >= g.nz ? gz - g.nz : gz);
        // (far outside a thin grid only behind its own halo: never read)
        if (gx >= g.nx || gy >= g.ny || gz >= g.nz) continue;
        const double v = src[((int64_t)gz * g.ny + gy) * g.nx + gx];
        const int l = ez * PXY + ey * PX + ex;
        A[0][l] = v;
        A[1][l] = v;
      }
      if (tid < 3) map[tid] = 0u;
      if (tid == 3) faces = 0u;
      __syncthreads();
      double d = owned ? A[0][at] : 0.0;  // a source keeps 0; so does a thread without a voxel
      const double d0 = d;
      unsigned int m = ~0u, all = 0u;
      int third = 0;  // sub mod 3
      for (int sub = 0; sub < max_sub; ++sub) {
        if (m & near) {
          const double *in = A[sub & 1];
          bool c = false;
          if (d != 0.0) {
            const double ax = fmin(in[at - 1], in[at + 1]);
            const double ay = fmin(in[at - PX], in[at + PX]);
            const double az = fmin(in[at - PXY], in[at + PXY]);
            if (fmin(fmin(ax, ay), az) < d) {
              const double v = godunov<ISO>(ax, ay, az, g);
              c = v < d && v <= g.rc_grid;
              d = c ? v : d;
            }
          }
          // (a block that did not change in the last sub-wave has its values
          // in both copies already)
          if (owned) A[(sub & 1) ^ 1][at] = d;
          if (__ballot(c) && lane == 0) atomicOr(&map[third], 1u << wave);
        }
        const int next = third == 2 ? 0 : third + 1;
        // read last two sub-waves ago, written from the next one on
        if (tid == 0) map[next] = 0u;
        __syncthreads();
        m = (unsigned int)__builtin_amdgcn_readfirstlane((int)map[third]);
        if (m == 0u) break;
        all |= m;
        third = next;
      }
      // both buffers hold an unchanged tile's values already if it did not
      // change in the last launch either
      if (owned && (all || prev))
        dst[((int64_t)(z0 + lz) * g.ny + (y0 + ly)) * g.nx + x0 + lx] = d;
      if (all) {
        any_changed = true;
        const bool c = d != d0;
        const int ex = min(TX, g.nx - x0) - 1, ey = min(TY, g.ny - y0) - 1,
                  ez = min(TZ, g.nz - z0) - 1;
        const unsigned int f = (__ballot(c && lx == 0) ? 1u : 0u) |
                               (__ballot(c && lx == ex) ? 2u : 0u) |
                               (__ballot(c && ly == 0) ? 4u : 0u) |
                               (__ballot(c && ly == ey) ? 8u : 0u) |
                               (__ballot(c && lz == 0) ? 16u : 0u) |
                               (__ballot(c && lz == ez) ? 32u : 0u);
        if (f && lane == 0) atomicOr(&faces, f);
        __syncthreads();
        if (tid == 0) w.changed[t] = (uint32_t)launch;
        if (tid < 7 && ((faces | 64u) >> tid & 1u)) {
          const int n = near_tile(w, tx, ty, tz, tid);
          const uint32_t next = (uint32_t)launch + 1u;
          if (w.live[n] && atomicMax(&w.stamp[n], next) != next)
            __hip_atomic_store(&w.list[next & 1][atomicAdd(&w.count[next], 1u)], n,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      if constexpr (TAIL) __threadfence();  // the tile's stores, before it counts as finished
      __syncthreads();  // the last map has been read before the next tile clears it
      if constexpr (TAIL)
        if (tid == 0) atomicAdd(&w.done[launch], 1u);
    }
    if (tid == 0 && any_changed)
      __hip_atomic_store(&flags[launch], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (TAIL) {
      if (tid == 0) {
        unsigned spins = 0;
        while (agent_load(&w.done[launch]) < (uint32_t)entries && ++spins < kTailSpins)
          __builtin_amdgcn_s_sleep(8);
        gave_up = spins == kTailSpins;
        if (gave_up)
          __hip_atomic_store(&flags[last], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      if (gave_up) return;
      __threadfence();  // the others' stores of this pass are read from here on
      __syncthreads();  // gave_up has been read
    }
  }
}

// ------------------------------------------------------------- plain waves
// Wave w reads state w-1 from buf[(w-1)&1] and writes state w to buf[w&1].
__global__ __launch_bounds__(256) void k_fsm_wave(double *dA, double *dB, SweepGeom g, int wave,
                                                  uint32_t *flags) {
  if (wave > 1 && flags[wave - 1] == 0u) return;
  const double *__restrict__ src = (wave & 1) ? dA : dB;
  double *__restrict__ dst = (wave & 1) ? dB : dA;
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
  bool chg = false;
  if (i < g.nx && j < g.ny) {
    const int im = i == 0 ? g.nx - 1 : i - 1, ip = i + 1 == g.nx ? 0 : i + 1;
    const int jm = j == 0 ? g.ny - 1 : j - 1, jp = j + 1 == g.ny ? 0 : j + 1;
    for (int k = blockIdx.z; k < g.nz; k += gridDim.z) {
      const int km = k == 0 ? g.nz - 1 : k - 1, kp = k + 1 == g.nz ? 0 : k + 1;
      const int64_t rowk = (int64_t)k * g.ny;
      const int64_t v = (rowk + j) * g.nx + i;
      const double d = src[v];
      if (d == 0.0) continue;
      const double ax = fmin(src[(rowk + j) * g.nx + im], src[(rowk + j) * g.nx + ip]);
      const double ay = fmin(src[(rowk + jm) * g.nx + i], src[(rowk + jp) * g.nx + i]);
      const double az = fmin(src[((int64_t)km * g.ny + j) * g.nx + i],
                             src[((int64_t)kp * g.ny + j) * g.nx + i]);
      const double gv = godunov<false>(ax, ay, az, g);
      const double nd = (gv < d && gv <= g.rc_grid) ? gv : d;
      dst[v] = nd;
      chg |= (nd != d);
    }
  }
  if (__syncthreads_or(chg ? 1 : 0) && threadIdx.x == 0) flags[wave] = 1u;
}

// The last pass is the first one that changed nothing (its output equals its
// input); if every pass changed something the sweep did not converge.
__global__ __launch_bounds__(256) void k_fsm_final(const double *dA, const double *dB,
                                                   int64_t nvox, double rc_grid,
                                                   const uint32_t *flags, int max_steps,
                                                   double *__restrict__ dist, int32_t *waves_out,
                                                   uint32_t *status) {
  const int last = sweep_last_pass(flags, max_steps);
  const double *__restrict__ D = (last & 1) ? dB : dA;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nvox;
       v += (int64_t)gridDim.x * blockDim.x) {
    double d = D[v];
    dist[v] = d > rc_grid ? rc_grid : d;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (waves_out) *waves_out = (int32_t)last;
    if (flags[max_steps] != 0u) atomicOr(status, ST_NOT_CONVERGED);
  }
}

static unsigned flat_grid(int64_t nvox) {
  int64_t b = ceil_div(nvox, 256 * 4);
  if (b < 1) b = 1;
  if (b > 4096) b = 4096;
  return (unsigned)b;
}

static SweepGeom geom(const int32_t nv[3], const double h[3], double rc_grid) {
  SweepGeom g;
  g.nx = nv[0];
  g.ny = nv[1];
  g.nz = nv[2];
  for (int k = 0; k < 3; ++k) {
    g.h[k] = h[k];
    g.w[k] = 1.0 / (h[k] * h[k]);
  }
  for (int k = 0; k < 3; ++k) {
    g.a2[k] = g.w[(k + 1) % 3] + g.w[(k + 2) % 3];
    g.a3[k] = g.a2[k] + g.w[k];
    g.r2[k] = 1.0 / g.a2[k];
    g.r3[k] = 1.0 / g.a3[k];
  }
  g.rc_grid = rc_grid;
  return g;
}

// The tiles' scratch: stamp, changed, the two lists (4 bytes a tile each),
// first and live (1 byte each).  The flags' scratch, max_steps + 2 words each:
// pass flags, list counts, entries taken, entries finished.
int64_t fsm_tile_bytes(const int32_t nv[3]) { return 18 * fsm_tile_count(nv); }
int64_t fsm_flag_words(int max_steps) { return 4 * ((int64_t)max_steps + 2); }

static SweepTiles sweep_tiles(const int32_t nv[3], void *tiles, uint32_t *flags, int max_steps) {
  SweepTiles w;
  w.ntx = (int)ceil_div(nv[0], TX);
  w.nty = (int)ceil_div(nv[1], TY);
  w.ntz = (int)ceil_div(nv[2], TZ);
  const int64_t n = fsm_tile_count(nv);
  w.stamp = static_cast<uint32_t *>(tiles);
  w.changed = w.stamp + n;
  w.list[0] = reinterpret_cast<int32_t *>(w.changed + n);
  w.list[1] = w.list[0] + n;
  w.first = reinterpret_cast<const uint8_t *>(w.list[1] + n);
  w.live = w.first + n;
  w.count = flags + max_steps + 2;
  w.taken = w.count + max_steps + 2;
  w.done = w.taken + max_steps + 2;
  return w;
}

static FsmInit init_args(const int32_t nv[3], bool tiled, double *dA, double *dB, void *tiles,
                         uint32_t *flags, int max_steps, dim3 *grid) {
  const int64_t nbx = ceil_div(nv[0], kInitX);
  *grid = dim3((unsigned)(nbx * ceil_div(nv[1], TY) * ceil_div(nv[2], TZ)));
  const SweepTiles w = sweep_tiles(nv, tiles, flags, max_steps);
  return FsmInit{nv[0], nv[1], nv[2], w.ntx, w.nty, (int)nbx, dA, dB,
                 tiled ? const_cast<uint8_t *>(w.first) : nullptr, const_cast<uint8_t *>(w.live),
                 w.stamp, w.changed, flags, (int)fsm_flag_words(max_steps)};
}

void launch_fsm_init(hipStream_t s, const uint8_t *seg, const uint8_t *iface, const int32_t nv[3],
                     bool tiled, double *dA, double *dB, void *tiles, uint32_t *flags,
                     int max_steps) {
  dim3 grid;
  const FsmInit p = init_args(nv, tiled, dA, dB, tiles, flags, max_steps, &grid);
  hipLaunchKernelGGL(k_fsm_init, grid, dim3(256), 0, s, seg, iface, p);
}

void launch_fsm_init_bits(hipStream_t s, const uint32_t *const maps[2], const Ctl *ctl,
                          const int32_t nv[3], bool tiled, double *dA, double *dB, void *tiles,
                          uint32_t *flags, int max_steps) {
  dim3 grid;
  const FsmInit p = init_args(nv, tiled, dA, dB, tiles, flags, max_steps, &grid);
  hipLaunchKernelGGL(k_fsm_init_bits, grid, dim3(256), 0, s, maps[0], maps[1], ctl, p);
}

// Workgroups of a tiled pass, each walking tiles in turn: one per compute unit.
// Two share its units without gaining on latency (and crowd the cell build that
// runs beside a step's sweep): with 512 and 256, ms per step of the 2.6 million
// slab 1.755 and 1.710, of the cylinder 0.975 and 0.934, of the droplet 0.425
// and 0.418.
constexpr int64_t kFsmTileBlocks = 256;
// and of the launch that goes on with several passes, few tiles each by then:
// more only wait (31 passes along a cylinder of 480 x 36 x 36 voxels, the last 17
// in that launch: one workgroup 3245 us, 32 1142, 128 and 256, with eight passes
// of their own, 1785 and 2836 against 1415)
constexpr int64_t kFsmTailBlocks = 32;
// From some thousands of tiles on what the list saves of a first pass comes near
// its launch (sweep without and with it: droplet, 2048 tiles 253 and 211 us, 4000
// 322 and 300, 5324 342 and 315, 10976 535 and 514; slab, 4000 125 and 129, 10000
// 567 and 576 with detection; gyroid, 4000 1313 and 1305, 6912 1635 and 1695).
constexpr int64_t kFsmListedTiles = 4096;

// Sub-waves of a pass.  settle: until the tile has settled, at most
// kSettleSubWaves.  Else the first kShortPasses passes take kShortSubWaves:
// with its halo frozen, most of what a tile does later in these is undone by
// its neighbours.  Corrections of the last digits then creep along a
// cylinder's axis, some 150 voxels, and settled passes take them a tile at a
// time.  (CPU model, passes and sub-waves of the slowest tiles: droplet
// settled 6 and 105, 8 in the first four 8 and 67, 4 throughout 11 and 41;
// cylinder 11 and 207, 13 and 186, 39 and 151.  8 x 8 x 8 tiles gain 8% of the
// droplet's step and need 20 passes for the cylinder.)
constexpr int kShortPasses = 4;
constexpr int kShortSubWaves = 8;
constexpr int kSettleSubWaves = 64;

void launch_fsm_step(hipStream_t s, double *dA, double *dB, void *tiles, const int32_t nv[3],
                     bool tiled, bool settle, const double h[3], double rc_grid, int step,
                     int last, uint32_t *flags, int max_steps) {
  const SweepGeom g = geom(nv, h, rc_grid);
  if (tiled) {
    const SweepTiles w = sweep_tiles(nv, tiles, flags, max_steps);
    int64_t blocks = fsm_tile_count(nv);
    const bool tail = last > step;
    blocks = std::min(blocks, tail ? kFsmTailBlocks : kFsmTileBlocks);
    const int subs = settle || step > kShortPasses ? kSettleSubWaves : kShortSubWaves;
    // The list pays its launch (5 us) while a workgroup's share of the tiles is
    // small: first pass of 1,800 tiles (droplet) 36 -> 18 us, 2,197 (cylinder)
    // 36 -> 32; of 10,000 (slab) 35 -> 31, less than its cost.
    const int64_t tiles_n = fsm_tile_count(nv);
    const bool listed = step == 1 && tiles_n > kFsmTileBlocks && tiles_n <= kFsmListedTiles;
    if (listed)
      hipLaunchKernelGGL(k_fsm_first, dim3((unsigned)ceil_div(tiles_n, 256)),
                         dim3(256), 0, s, w);
    const bool iso = h[0] == h[1] && h[1] == h[2];
    const auto kernel = iso ? (tail ? k_fsm_tiles<true, true> : k_fsm_tiles<true, false>)
                            : (tail ? k_fsm_tiles<false, true> : k_fsm_tiles<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kTileThreads), 0, s, dA, dB, w, g, step,
                       last, listed, subs, flags);
  } else {
    int zb = nv[2] < 64 ? nv[2] : 64;
    hipLaunchKernelGGL(k_fsm_wave,
                       dim3((unsigned)ceil_div(nv[0], 64), (unsigned)ceil_div(nv[1], 4),
                            (unsigned)zb),
                       dim3(256), 0, s, dA, dB, g, step, flags);
  }
}

void launch_fsm_final(hipStream_t s, const double *dA, const double *dB, int64_t nvox,
                      double rc_grid, const uint32_t *flags, int max_steps, double *dist,
                      int32_t *waves_out, uint32_t *status) {
  hipLaunchKernelGGL(k_fsm_final, dim3(flat_grid(nvox)), dim3(256), 0, s, dA, dB, nvox,
                     rc_grid, flags, max_steps, dist, waves_out, status);
}

}  // namespace dcm
