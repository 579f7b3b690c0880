// Cutoff assignment (Section 2.2) and linked-cell binning (Section 2.3).
#include "cells_device.hpp"

namespace dcm {

// ----------------------------------------------------- cutoff assignment
// delta_i: periodic trilinear interpolation of the voxel-centred distances at
// the particle; rc_i = rc_max - (rc_max - rc_min) * min(delta_i/ramp, 1).
// SWEEP: D is the sweep's own pair of buffers (D, D2) and its pass flags,
// read as the sweep's final pass would write the field: the buffer of the
// first pass that changed nothing, each value capped at `cap`; a sweep that
// ran out of passes is flagged here.
// SLOTS: cells built before the cutoffs were known (their records carry no
// cutoff): the threads walk the sorted slots, particle p = perm[slot], and
// each record takes its particle's cutoff, clamped to [0, rc_cap] as the
// cell build's gather clamps it (a value outside is flagged).
template <bool SWEEP>
struct CutoffField {
  const double *D;
  int nx, ny, nz;
  double Lx, Ly, Lz, sx, sy, sz, rc_min, rc_max, ramp, cap;

  // the field's buffer (SWEEP), once per workgroup
  __device__ __forceinline__ explicit CutoffField(const CutoffArgs &a)
      : D(a.D), nx(a.nv[0]), ny(a.nv[1]), nz(a.nv[2]), Lx(a.L[0]), Ly(a.L[1]), Lz(a.L[2]),
        sx(a.sc[0]), sy(a.sc[1]), sz(a.sc[2]), rc_min(a.rule.rc_min), rc_max(a.rule.rc_max),
        ramp(a.rule.ramp), cap(a.cap) {
    if constexpr (SWEEP) {
      if (sweep_last_pass(a.flags, a.max_steps) & 1) D = a.D2;
      if (blockIdx.x == 0 && threadIdx.x == 0 && a.flags[a.max_steps] != 0u)
        atomicOr(a.status, ST_NOT_CONVERGED);
    }
  }

  // cutoff of a particle (rc_max if its position is not finite), and its delta
  __device__ __forceinline__ double at(double px, double py, double pz, double &delta) const {
    if (!finite3(px, py, pz)) {
      delta = __builtin_nan("");
      return rc_max;
    }
    const double pos[3] = {wrap_coord(px, Lx), wrap_coord(py, Ly), wrap_coord(pz, Lz)};
    const double sc[3] = {sx, sy, sz};
    const int nn[3] = {nx, ny, nz};
    int i0[3], i1[3];
    double t[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double u = pos[a] * sc[a] - 0.5;
      double f = floor(u);
      t[a] = u - f;
      int ia = (int)f;  // f lies in [-1, n)
      i0[a] = ia < 0 ? ia + nn[a] : ia;
      i1[a] = ia + 1 >= nn[a] ? ia + 1 - nn[a] : ia + 1;
    }
    auto DV = [&](int i, int j, int k) {
      const double v = D[((int64_t)k * ny + j) * nx + i];
      if constexpr (SWEEP) return v > cap ? cap : v;
      else return v;
    };
    double wx0 = 1.0 - t[0], wx1 = t[0];
    double wy0 = 1.0 - t[1], wy1 = t[1];
    double wz0 = 1.0 - t[2], wz1 = t[2];
    double c00 = DV(i0[0], i0[1], i0[2]) * wx0 + DV(i1[0], i0[1], i0[2]) * wx1;
    double c10 = DV(i0[0], i1[1], i0[2]) * wx0 + DV(i1[0], i1[1], i0[2]) * wx1;
    double c01 = DV(i0[0], i0[1], i1[2]) * wx0 + DV(i1[0], i0[1], i1[2]) * wx1;
    double c11 = DV(i0[0], i1[1], i1[2]) * wx0 + DV(i1[0], i1[1], i1[2]) * wx1;
    double c0 = c00 * wy0 + c10 * wy1;
    double c1 = c01 * wy0 + c11 * wy1;
    delta = c0 * wz0 + c1 * wz1;
    double q = delta / ramp;
    if (q > 1.0) q = 1.0;
    return rc_max - (rc_max - rc_min) * q;
  }
};

template <bool SWEEP, bool SLOTS>
__global__ __launch_bounds__(256) void k_assign_cutoffs(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    int64_t n, CutoffArgs a, const int32_t *__restrict__ perm, double4 *__restrict__ sorted,
    double rc_cap) {
  const CutoffField<SWEEP> field(a);
  for (int64_t it = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; it < n;
       it += (int64_t)gridDim.x * blockDim.x) {
    int64_t p = it;
    if constexpr (SLOTS) p = perm[it];
    double d;
    const double r = field.at(x[p], y[p], z[p], d);
    if (a.delta) a.delta[p] = d;
    a.rc[p] = r;
    if constexpr (SLOTS) {  // the record's cutoff as the gather writes it
      if (!(r >= 0.0) || r > rc_cap) atomicOr(a.status, ST_RC_RANGE);
      sorted[it].w = (r >= 0.0) ? (r < rc_cap ? r : rc_cap) : 0.0;  // NaN -> 0
    }
  }
}

void launch_assign_cutoffs(hipStream_t s, const double *x, const double *y, const double *z,
                           int64_t n, const CutoffArgs &a, const int32_t *perm, double4 *sorted,
                           double rc_cap) {
  if (n <= 0) return;
  int64_t b = ceil_div(n, 256);
  if (b > 16384) b = 16384;
  if (perm)
    hipLaunchKernelGGL((k_assign_cutoffs<true, true>), dim3((unsigned)b), dim3(256), 0, s, x, y,
                       z, n, a, perm, sorted, rc_cap);
  else if (a.flags)
    hipLaunchKernelGGL((k_assign_cutoffs<true, false>), dim3((unsigned)b), dim3(256), 0, s, x, y,
                       z, n, a, nullptr, nullptr, 0.0);
  else
    hipLaunchKernelGGL((k_assign_cutoffs<false, false>), dim3((unsigned)b), dim3(256), 0, s, x, y,
                       z, n, a, nullptr, nullptr, 0.0);
}

// ------------------------------------------------------------ cell count
// ASSIGN: the cutoffs are assigned here, from the sweep's field, instead of
// read: the positions are in registers, and a launch is saved (4.6 + 4.7 us
// apart, 5.0 in one at 20,000 particles; 17 + 22 and 31 us at 1.2 million).
template <bool ASSIGN>
__global__ __launch_bounds__(256) void k_cell_count(
    CutoffArgs cut, const double *__restrict__ x, const double *__restrict__ y,
    const double *__restrict__ z, const double *__restrict__ rc, int64_t n, double Lx, double Ly,
    double Lz, int nx, int ny, int nz, double sx, double sy, double sz, double rc_cap,
    int32_t *__restrict__ cell_of, int32_t *__restrict__ slot, int32_t *count,
    unsigned long long *__restrict__ block_max, uint32_t *__restrict__ xq, Ctl *ctl,
    uint32_t *status) {
  const CutoffField<ASSIGN> field(cut);
  unsigned long long rmax = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->big_cells = 0u;  // for the cell sort that follows
  // uniform trip count: every lane reaches the run-aggregated atomic
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t base = blockIdx.x * (int64_t)blockDim.x; base < n; base += stride) {
    const int64_t i = base + threadIdx.x;
    const bool valid = i < n;
    int c = 0;
    if (valid) {
      // rc null: the cutoffs are not known yet (the cutoff assignment adds them)
      double px = x[i], py = y[i], pz = z[i], r = 0.0;
      if constexpr (ASSIGN) {
        double d;
        r = field.at(px, py, pz, d);
        if (cut.delta) cut.delta[i] = d;
        cut.rc[i] = r;
      } else if (rc) {
        r = rc[i];
      }
      uint32_t q = 0;
      if (finite3(px, py, pz)) {
        const double wx = wrap_coord(px, Lx);
        int cx = slab_index(wx, sx, nx);
        int cy = slab_index(wrap_coord(py, Ly), sy, ny);
        int cz = slab_index(wrap_coord(pz, Lz), sz, nz);
        c = (cz * ny + cy) * nx + cx;
        q = x_key(wx, sx, cx);
      } else {
        atomicOr(status, ST_NONFINITE_POS);
      }
      if (xq) xq[i] = q;
      // rc_cap: the build's bound on every cutoff (inclusive, below L/2)
      if (!(r >= 0.0) || r > rc_cap) {
        atomicOr(status, ST_RC_RANGE);
        r = (r > rc_cap) ? rc_cap : 0.0;
      }
      unsigned long long bits = (unsigned long long)__double_as_longlong(r);
      rmax = bits > rmax ? bits : rmax;
      cell_of[i] = c;
    }
    // the counter's value before is the particle's slot in its cell
    const int sl = wave_run_slot(count, (uint32_t)c, valid);
    if (valid) slot[i] = sl;
  }
  // the workgroup's largest cutoff, stored without atomics (one address
  // shared by every workgroup would serialise them)
  __shared__ unsigned long long wmax[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    unsigned long long o = __shfl_xor(rmax, off, 64);
    rmax = o > rmax ? o : rmax;
  }
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = rmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = wmax[0];
    for (int w = 1; w < 4; ++w) m = wmax[w] > m ? wmax[w] : m;
    block_max[blockIdx.x] = m;
  }
}

int64_t cell_count_blocks(int64_t n) {
  int64_t b = ceil_div(n, 256);
  if (b > 16384) b = 16384;
  return b < 1 ? 1 : b;
}

void launch_cell_count(hipStream_t s, const double *x, const double *y, const double *z,
                       const double *rc, int64_t n, const double L[3], const int32_t nc[3],
                       const double sc[3], double rc_cap, int32_t *cell_of, int32_t *slot,
                       int32_t *cell_count, unsigned long long *block_max, uint32_t *xq, Ctl *ctl,
                       uint32_t *status, const CutoffArgs *assign) {
  if (n <= 0) return;
  const dim3 g((unsigned)cell_count_blocks(n)), b(256);
  if (assign)
    hipLaunchKernelGGL(k_cell_count<true>, g, b, 0, s, *assign, x, y, z, rc, n, L[0], L[1], L[2],
                       nc[0], nc[1], nc[2], sc[0], sc[1], sc[2], rc_cap, cell_of, slot,
                       cell_count, block_max, xq, ctl, status);
  else
    hipLaunchKernelGGL(k_cell_count<false>, g, b, 0, s, CutoffArgs{}, x, y, z, rc, n, L[0], L[1],
                       L[2], nc[0], nc[1], nc[2], sc[0], sc[1], sc[2], rc_cap, cell_of, slot,
                       cell_count, block_max, xq, ctl, status);
}

// ------------------------------------------------------- exclusive scan
int64_t scan_tmp_elems(int64_t n) { return ceil_div(n, kScanTile) + 1; }

__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const int32_t *__restrict__ in,
                                                             int64_t n, int32_t *tile_sum) {
  __shared__ int32_t lds[kScanThreads / 64];
  const int64_t base = blockIdx.x * (int64_t)kScanTile + threadIdx.x * kScanPer;
  int32_t v[kScanPer];
  load_run(in, base, n, v);
  int32_t s = 0;
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) s += v[q];
  int32_t total;
  block_exclusive_scan<kScanThreads / 64>(s, lds, &total);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// Exclusive scan of the tile totals in place; each thread owns a run of
// consecutive tiles.
__global__ __launch_bounds__(kTotalsThreads) void k_scan_totals(int32_t *tile_sum, int64_t ntiles,
                                                                int32_t *out_last) {
  __shared__ int32_t lds[kTotalsThreads / 64];
  const int64_t per = (ntiles + kTotalsThreads - 1) / kTotalsThreads;
  const int64_t t0 = threadIdx.x * per;
  const int64_t t1 = t0 + per < ntiles ? t0 + per : ntiles;
  int32_t s = 0;
  for (int64_t t = t0; t < t1; ++t) s += tile_sum[t];
  int32_t total;
  int32_t run = block_exclusive_scan<kTotalsThreads / 64>(s, lds, &total);
  for (int64_t t = t0; t < t1; ++t) {
    const int32_t v = tile_sum[t];
    tile_sum[t] = run;
    run += v;
  }
  if (threadIdx.x == 0) *out_last = total;
}

// Each tile's local scan plus its offset: the scanned tile totals (SUM
// false), or the sum of the raw totals of the tiles before it (SUM true: no
// separate pass over the totals; the last tile also writes out[n]).
template <bool SUM>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const int32_t *in, int64_t n,
                                                             const int32_t *__restrict__ tile_off,
                                                             int32_t *__restrict__ out,
                                                             ScanClear clr) {
  __shared__ int32_t lds[kScanThreads / 64];
  int32_t off;
  if constexpr (SUM) {
    int32_t pre = 0;
    for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kScanThreads) pre += tile_off[t];
    block_exclusive_scan<kScanThreads / 64>(pre, lds, &off);
  } else {
    off = tile_off[blockIdx.x];
  }
  const int64_t base = blockIdx.x * (int64_t)kScanTile + threadIdx.x * kScanPer;
  int32_t v[kScanPer];
  load_run(in, base, n, v);
  int32_t s = 0;
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) s += v[q];
  int32_t total;
  const int32_t run = block_exclusive_scan<kScanThreads / 64>(s, lds, &total) + off;
  if (SUM && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = off + total;
  store_run(out, base, n, v, run, clr);
}

__global__ __launch_bounds__(kTotalsThreads) void k_scan_one(const int32_t *in, int64_t n,
                                                             int32_t *out, ScanClear clr) {
  __shared__ int32_t lds[kTotalsThreads / 64];
  scan_by_block<kTotalsThreads>(in, n, out, lds, clr);
}

// Up to this many elements one workgroup scans in one launch, in one round
// (4.6 us traced against 4.1 + 4.3 for two launches; two rounds take 10.7).
constexpr int64_t kScanOneMax = (int64_t)kTotalsThreads * kScanPer;

static void launch_scan(hipStream_t s, const int32_t *in, int32_t *out, int64_t n, int32_t *tmp,
                        const ScanClear &clr) {
  // out has n + 1 entries; out[n] = total.  in, out and the cleared arrays are
  // 16-byte aligned.
  if (n <= kScanOneMax) {
    hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(kTotalsThreads), 0, s, in, n, out, clr);
    return;
  }
  const int64_t ntiles = ceil_div(n, kScanTile);
  hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, in, n, tmp);
  if (ntiles <= kScanSumTiles) {
    // each tile sums the totals before it (at most kScanSumTiles / 256 reads
    // per thread): two launches
    hipLaunchKernelGGL(k_scan_apply<true>, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, in,
                       n, tmp, out, clr);
    return;
  }
  hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(kTotalsThreads), 0, s, tmp, ntiles, out + n);
  hipLaunchKernelGGL(k_scan_apply<false>, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, in, n,
                     tmp, out, clr);
}

void launch_exclusive_scan(hipStream_t s, const int32_t *in, int32_t *out, int64_t n,
                           int32_t *tmp) {
  launch_scan(s, in, out, n, tmp, ScanClear{nullptr, nullptr});
}

void launch_cell_scan(hipStream_t s, int32_t *cell_count, int32_t *cell_start, int64_t ncell,
                      uint32_t *qword, int32_t *tmp) {
  launch_scan(s, cell_count, cell_start, ncell, tmp, ScanClear{cell_count, qword});
}

// ------------------------------------------------ scatter + stable order
// Every particle to its slot (the count's): perm[slot] = id, skey[slot] = its x
// key.  The first row_blocks workgroups instead form the extended rows' counts
// (one thread per row), which also need only the cell starts, and the last one
// the largest cutoff from the count's maxima per workgroup.
struct ExtRows {
  ExtGeom g;
  int64_t nrows;
  int32_t *row_count, *row_lo;
};
__device__ __forceinline__ void reduce_rcmax(const unsigned long long *__restrict__ bm, int nb,
                                             Ctl *ctl) {
  __shared__ unsigned long long wmax[4];
  unsigned long long m = 0;
#pragma unroll 8
  for (int b = threadIdx.x; b < nb; b += 256) m = bm[b] > m ? bm[b] : m;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    unsigned long long o = __shfl_xor(m, off, 64);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 0; w < 4; ++w) m = wmax[w] > m ? wmax[w] : m;
    ctl->rc_max_bits = m;
  }
}
__global__ __launch_bounds__(256) void k_cell_scatter(const int32_t *__restrict__ cell_of,
                                                      const int32_t *__restrict__ slot, int64_t n,
                                                      const int32_t *__restrict__ cell_start,
                                                      int32_t *__restrict__ perm,
                                                      const uint32_t *__restrict__ xq,
                                                      uint32_t *__restrict__ skey,
                                                      unsigned row_blocks, ExtRows rows,
                                                      const unsigned long long *__restrict__ bm,
                                                      int nmax, Ctl *ctl) {
  if (blockIdx.x == gridDim.x - 1) {
    reduce_rcmax(bm, nmax, ctl);
    return;
  }
  if (blockIdx.x < row_blocks) {
    const int row = (int)(blockIdx.x * 256 + threadIdx.x);
    if (row < (int)rows.nrows)
      rows.row_count[row] = ext_row_count(cell_start, rows.g, row, rows.row_lo[row]);
    return;
  }
  const int64_t stride = (int64_t)(gridDim.x - 1 - row_blocks) * blockDim.x;
  for (int64_t i = (blockIdx.x - row_blocks) * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += stride) {
    const int64_t p = cell_start[cell_of[i]] + slot[i];
    perm[p] = (int32_t)i;
    skey[p] = xq[i];
  }
}

// One thread per slot of the cell-scattered order perm (x keys skey): a
// particle of a small cell moves to its cell's start plus its rank there
// (the count of the cell's particles with smaller (x key, id)); a particle
// of a large cell keeps its slot.  out receives the result; no thread waits
// on another.
// A particle of a small cell also writes its sorted record at its final slot
// (no gather pass of its own).  The thread of a cell's first slot writes the
// cell's sub-cell word (cells without particles keep the 0 that the scan of the
// counts left), and lists a cell too large to rank.
// SCAN: the first workgroup instead scans the extended rows' counts, beside
// the others' work.
template <bool SCAN>
__global__ __launch_bounds__(256) void k_cell_rank(const int32_t *__restrict__ cell_start,
                                                   const int32_t *__restrict__ cell_of,
                                                   const int32_t *__restrict__ perm, int64_t n,
                                                   const uint32_t *__restrict__ skey,
                                                   uint32_t *__restrict__ qword,
                                                   int32_t *__restrict__ out,
                                                   int32_t *__restrict__ big_list,
                                                   uint32_t *big_count, GatherOut go,
                                                   const int32_t *__restrict__ row_count,
                                                   int64_t nrows, int32_t *__restrict__ row_start) {
  if constexpr (SCAN) {
    __shared__ int32_t lds[256 / 64];
    if (blockIdx.x == 0) {
      scan_by_block<256>(row_count, nrows, row_start, lds, ScanClear{nullptr, nullptr});
      return;
    }
  }
  const unsigned skip = SCAN ? 1u : 0u;
  for (int64_t p = (blockIdx.x - skip) * (int64_t)blockDim.x + threadIdx.x; p < n;
       p += (int64_t)(gridDim.x - skip) * blockDim.x) {
    const int i = perm[p];
    // the record's inputs are read while the cell's keys are counted
    const double px = go.x[i], py = go.y[i], pz = go.z[i], pr = go.rc ? go.rc[i] : 0.0;
    const int c = cell_of[i];
    const int a = cell_start[c], b = cell_start[c + 1];
    if (p == a) {
      if (qword) qword[c] = sub_word(skey, a, b);
      if (b - a > kSmallCell) big_list[atomicAdd(big_count, 1u)] = (int32_t)c;
    }
    if (b - a > kSmallCell) {
      out[p] = i;
      continue;
    }
    const int r = rank_in_cell(perm, skey, p, i, a, b);
    out[a + r] = i;
    go.sorted[a + r] = gather_record(go.L, go.rc_cap, px, py, pz, pr);
  }
}

int64_t cell_sort_list_elems(int64_t n) { return n / (kSmallCell + 1) + 1; }

// ------------------------------------------------ periodic ghost images
// The extended grid (ExtGeom) lets a lane walk any row of cells around its
// particle as one contiguous range of the extended array, without
// wrap-around or image shifts.
//
// It is built row by row.  An extended row (ey, ez) repeats real row
// (ry, rz) periodically along x.  With S(r) the particles of the real row in
// its cells [0, r) and T its total, the particles in unwrapped cells [0, u)
// number F(u) = p T + S(r) for u = p n_x + r, 0 <= r < n_x, and the extended
// row holds unwrapped cells [-h_x, n_x + h_x): its k-th particle is the
// unwrapped particle P = F(-h_x) + k, i.e. particle P mod T of the real row
// shifted by floor(P / T) periods.

// ext_start of every extended cell (and of one past the last) from the row
// starts, one wavefront per extended row with the row's values uniform.  Cell
// u of the unwrapped row lies p = floor(u / n_x) periods away; with a halo of
// at most n_x cells, u is in [-n_x, 2 n_x) and p in {-1, 0, 1}.
// The last big_blocks workgroups instead sort the cells too large to rank.
// host_total (pinned, null: none) receives the extended count as well: read
// by the host once the launch is complete, without a copy of its own.
__global__ __launch_bounds__(256) void k_ext_starts(
    const int32_t *__restrict__ cell_start, const int32_t *__restrict__ row_start,
    const int32_t *__restrict__ row_lo, ExtGeom g, int64_t next, int64_t nrows,
    int32_t *__restrict__ ext_start, const uint32_t *__restrict__ qword,
    int2 *__restrict__ ext_sq, int32_t *host_total, unsigned big_blocks, int32_t *perm,
    int32_t *tmp, const uint32_t *__restrict__ xq, const int32_t *__restrict__ big_list,
    const uint32_t *big_count, GatherOut go) {
  const unsigned own = gridDim.x - big_blocks;
  if (blockIdx.x >= own) {
    sort_big_cells(cell_start, perm, tmp, xq, big_list, big_count, blockIdx.x - own, big_blocks,
                   [&](int64_t, int slot, int id) { go.sorted[slot] = gather_record(go, id); });
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(
      (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6));
  const int nwaves = (int)(((int64_t)own * blockDim.x) >> 6);
  if (wave == 0 && lane == 0) {
    const int32_t total = row_start[nrows];
    ext_start[next] = total;
    if (ext_sq) ext_sq[next] = make_int2(total, 0);
    if (host_total)
      __hip_atomic_store(host_total, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  const int nx = g.nc[0], hx = g.h[0], nex = g.ne[0];
  const bool near = hx <= nx;
  // next < 2^30 (checked at build), so 32-bit cell indices suffice
  for (int row = wave; row < (int)nrows; row += nwaves) {
    const ExtRow r = ext_row(g, row);
    const int c0 = cell_start[r.r0];
    const int64_t T = cell_start[r.r0 + nx] - c0;
    const int64_t base = (int64_t)row_start[row] - row_lo[row];
    int32_t *__restrict__ out = ext_start + (int64_t)row * nex;
    for (int ex = lane; ex < nex; ex += 64) {
      const int u = ex - hx;
      const int p = near ? (u < 0 ? -1 : (u >= nx ? 1 : 0)) : floor_div(u, nx);
      const int rc = r.r0 + (u - p * nx);
      const int32_t st = (int32_t)(base + p * T + (cell_start[rc] - c0));
      out[ex] = st;
      if (ext_sq) ext_sq[(int64_t)row * nex + ex] = make_int2(st, (int)qword[rc]);
    }
  }
}

// Copy of every extended row, one wavefront per row.  Writes stop at the
// buffer's capacity; running past it flags an overflow (the pair kernel then
// refuses to read ghost ranges beyond the capacity).  Each of ext_pos,
// ext_rel and ext_src (the source's sorted slot) is written when not null.
__global__ __launch_bounds__(256) void k_ext_fill(const int32_t *__restrict__ cell_start,
                                                  const int32_t *__restrict__ row_start,
                                                  const int32_t *__restrict__ row_lo,
                                                  const double4 *__restrict__ sorted, ExtGeom g,
                                                  int64_t nrows, int64_t cap,
                                                  double4 *__restrict__ ext_pos,
                                                  float4 *__restrict__ ext_rel,
                                                  int32_t *__restrict__ ext_src,
                                                  uint32_t *status) {
  const double len[3] = {g.L[0] / (double)g.nc[0], g.L[1] / (double)g.nc[1],
                         g.L[2] / (double)g.nc[2]};
  const double sc0 = (double)g.nc[0] / g.L[0];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(
      (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6));
  const int nwaves = (int)(((int64_t)gridDim.x * blockDim.x) >> 6);
  // with a halo of at most n_x cells a row's unwrapped prefixes P lie in
  // [-T, 2T), so the period floor(P / T) is -1, 0 or 1
  const bool near = g.h[0] <= g.nc[0];
  for (int row = wave; row < (int)nrows; row += nwaves) {
    const ExtRow r = ext_row(g, row);
    const int first = cell_start[r.r0];
    const int T = cell_start[r.r0 + g.nc[0]] - first;
    const int64_t o0 = row_start[row], cnt = row_start[row + 1] - o0;
    const int lo = row_lo[row];
    const double sy = (double)r.py * g.L[1], sz = (double)r.pz * g.L[2];
    bool over = false;
    // kFillUnroll slots per lane at a time: their source reads are all
    // issued before the first is used
    constexpr int kFillUnroll = 4;
    for (int k0 = lane; k0 < cnt; k0 += 64 * kFillUnroll) {
      double4 q[kFillUnroll];
      int pk[kFillUnroll];
      bool ok[kFillUnroll];
#pragma unroll
      for (int u = 0; u < kFillUnroll; ++u) {
        const int k = k0 + 64 * u;
        const int P = lo + k;
        // cnt > 0 implies T > 0
        const int p = near ? (P < 0 ? -1 : (P >= T ? 1 : 0)) : floor_div(P, T);
        const int64_t o = o0 + k;
        pk[u] = p;
        ok[u] = k < cnt;
        if (ok[u] && o >= cap) {
          over = true;
          ok[u] = false;
        }
        const int src = first + (P - p * T);
        if (ok[u] && ext_src) ext_src[o] = src;
        if (ok[u] && ext_pos) q[u] = sorted[src];
      }
      if (!ext_pos) continue;
#pragma unroll
      for (int u = 0; u < kFillUnroll; ++u) {
        if (!ok[u]) continue;
        const int64_t o = o0 + k0 + 64 * u;
        const int p = pk[u];
        double4 w = q[u];
        const int ex = slab_index(w.x, sc0, g.nc[0]) + p * g.nc[0];
        w.x = w.x + (double)p * g.L[0];
        w.y = w.y + sy;
        w.z = w.z + sz;
        ext_pos[o] = w;
        if (ext_rel) ext_rel[o] = rel_record(w, ex, r.ey, r.ez, len);
      }
    }
    if (over) atomicOr(status, ST_GHOST_OVERFLOW);
  }
}

int64_t ext_row_scratch_elems(const int32_t nc[3], const int32_t h[3]) {
  return (int64_t)(nc[1] + 2 * h[1]) * (nc[2] + 2 * h[2]) + 1;
}

static ExtGeom ext_geom(const int32_t nc[3], const int32_t h[3], const double L[3]) {
  ExtGeom g;
  for (int a = 0; a < 3; ++a) {
    g.nc[a] = nc[a];
    g.h[a] = h[a];
    g.ne[a] = nc[a] + 2 * h[a];
    g.L[a] = L[a];
  }
  return g;
}

static void launch_ext_fill(hipStream_t s, const int32_t *cell_start, const int32_t *row_start,
                            const int32_t *row_lo, const double4 *sorted, const ExtGeom &g,
                            int64_t ext_cap, double4 *ext_pos, float4 *ext_rel,
                            int32_t *ext_src, uint32_t *status) {
  const int64_t nrows = (int64_t)g.ne[1] * g.ne[2];
  int64_t b = ceil_div(nrows, 4);  // four rows per workgroup of 256
  if (b > 16384) b = 16384;
  hipLaunchKernelGGL(k_ext_fill, dim3((unsigned)b), dim3(256), 0, s, cell_start, row_start,
                     row_lo, sorted, g, nrows, ext_cap, ext_pos, ext_rel, ext_src, status);
}

void launch_ext_src(hipStream_t s, const int32_t *cell_start, const int32_t *row_start,
                    const int32_t *row_lo, const int32_t nc[3], const int32_t h[3],
                    const double L[3], int64_t ext_cap, int32_t *ext_src, uint32_t *status) {
  launch_ext_fill(s, cell_start, row_start, row_lo, nullptr, ext_geom(nc, h, L), ext_cap, nullptr,
                  nullptr, ext_src, status);
}

void launch_ext_refill(hipStream_t s, const int32_t *cell_start, const int32_t *row_start,
                       const int32_t *row_lo, const double4 *sorted, const int32_t nc[3],
                       const int32_t h[3], const double L[3], int64_t ext_cap, double4 *ext_pos,
                       uint32_t *status) {
  launch_ext_fill(s, cell_start, row_start, row_lo, sorted, ext_geom(nc, h, L), ext_cap, ext_pos,
                  nullptr, nullptr, status);
}

// Seven launches a build: count, scan (one up to 16K cells, else two), scatter
// with the rows' counts and the largest cutoff, rank with the gather and the
// rows' scan, starts with the sort of large cells, fill.  Each of them takes
// 4-6 us below about 100,000 particles, whatever it does, so stages that wait
// for the same predecessor share a launch and no launch clears scratch memory:
// a whole step went from 1217 to 1082 us per ten steps of 20,000 particles
// (FP32-mixed), from 1974 to 1850 at 99,000 (FP64) and from 12089 to 11924 at
// 1.2 million.  At 2.6 million the count takes 55 us instead of 33 (its atomics
// return the slots) and the scatter 28 instead of 35, without its own atomics.
void launch_cell_order(hipStream_t s, const CellOrder &o) {
  const ExtGeom g = ext_geom(o.nc, o.h, o.L);
  const int64_t next = (int64_t)g.ne[0] * g.ne[1] * g.ne[2];
  const int64_t nrows = (int64_t)g.ne[1] * g.ne[2];
  const unsigned row_blocks = (unsigned)ceil_div(nrows, 256);
  const unsigned pblocks = (unsigned)std::min<int64_t>(ceil_div(o.n, 256), 16384);
  const ExtRows rows = {g, nrows, o.row_count, o.row_lo};
  hipLaunchKernelGGL(k_cell_scatter, dim3(row_blocks + pblocks + 1), dim3(256), 0, s,
                     o.cell_of, o.slot, o.n, o.cell_start, o.scratch, o.xq, o.skey, row_blocks,
                     rows, o.block_max, o.n > 0 ? (int)cell_count_blocks(o.n) : 0, o.ctl);
  const bool fused = o.n > 0 && nrows <= kRowScanMax;
  if (!fused) launch_exclusive_scan(s, o.row_count, o.row_start, nrows, o.scan_tmp);
  if (fused)
    hipLaunchKernelGGL(k_cell_rank<true>, dim3(pblocks + 1), dim3(256), 0, s, o.cell_start,
                       o.cell_of, o.scratch, o.n, o.skey, o.qword, o.perm, o.big_list,
                       o.big_count, o.go, o.row_count, nrows, o.row_start);
  else if (o.n > 0)
    hipLaunchKernelGGL(k_cell_rank<false>, dim3(pblocks), dim3(256), 0, s, o.cell_start,
                       o.cell_of, o.scratch, o.n, o.skey, o.qword, o.perm, o.big_list,
                       o.big_count, o.go, nullptr, 0, nullptr);
  // the large cells are sorted in place in perm, with the scatter's order as
  // scratch
  const unsigned big_blocks = o.n > kSmallCell ? (unsigned)kBigSortBlocks : 0u;
  const unsigned b = (unsigned)std::min<int64_t>(std::max<int64_t>(ceil_div(nrows, 4), 1), 16384);
  hipLaunchKernelGGL(k_ext_starts, dim3(b + big_blocks), dim3(256), 0, s, o.cell_start,
                     o.row_start, o.row_lo, g, next, nrows, o.ext_start, o.qword, o.ext_sq,
                     o.host_total, big_blocks, o.perm, o.scratch, o.xq, o.big_list, o.big_count,
                     o.go);
}

void launch_ext_images(hipStream_t s, const int32_t *cell_start, const int32_t *row_start,
                       const int32_t *row_lo, const double4 *sorted, const int32_t nc[3],
                       const int32_t h[3], const double L[3], int64_t ext_cap, double4 *ext_pos,
                       float4 *ext_rel, uint32_t *status) {
  launch_ext_fill(s, cell_start, row_start, row_lo, sorted, ext_geom(nc, h, L), ext_cap, ext_pos,
                  ext_rel, nullptr, status);
}

}  // namespace dcm
