// Device parts of the cell build that the single-system kernels (k_cells.hip)
// and the batched ones (k_batch.hip) share: the scan by one workgroup, the
// order of a cell's particles, its sub-cell word and the sort of large cells.
#pragma once

#include "dcm_device.hpp"
#include "dcm_internal.hpp"

namespace dcm {

// Three phases over tiles of kScanTile elements: tile totals, one workgroup
// scanning the totals, then each tile's local scan plus its offset.  A thread
// owns kScanPer consecutive elements, read and written as int4.
constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanTile = kScanThreads * kScanPer;
constexpr int kTotalsThreads = 1024;
constexpr int64_t kScanSumTiles = 4096;  // up to this many tiles: no pass over the totals

// Inclusive scan over the 64 lanes of a wavefront.
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}

// Exclusive scan over the workgroup (NW wavefronts); lds holds NW entries.
template <int NW>
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t *lds, int32_t *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int32_t incl = wave_inclusive_scan(v);
  if (lane == 63) lds[w] = incl;
  __syncthreads();
  int32_t before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    const int32_t t = lds[k];
    before += k < w ? t : 0;
    all += t;
  }
  __syncthreads();  // lds may be reused after this
  *total = all;
  return before + incl - v;
}

// this thread's kScanPer elements starting at base (zeros past n)
__device__ __forceinline__ void load_run(const int32_t *in, int64_t base, int64_t n,
                                         int32_t (&v)[kScanPer]) {
  if (base + kScanPer <= n) {
    const int4 *p = reinterpret_cast<const int4 *>(in + base);
#pragma unroll
    for (int q = 0; q < kScanPer / 4; ++q) {
      const int4 t = p[q];
      v[4 * q] = t.x;
      v[4 * q + 1] = t.y;
      v[4 * q + 2] = t.z;
      v[4 * q + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) v[q] = base + q < n ? in[base + q] : 0;
  }
}

// What a scan of per-cell counts leaves behind: the counts zeroed for the next
// build (which then needs no launch to clear them), and a second array of the
// same length zeroed (the sub-cell words, which the rank writes for the cells
// that hold particles).  Either null: not touched.
struct ScanClear {
  int32_t *counts;
  uint32_t *words;
};

// this thread's kScanPer elements starting at base, scanned from `run` on
__device__ __forceinline__ void store_run(int32_t *__restrict__ out, int64_t base, int64_t n,
                                          const int32_t (&v)[kScanPer], int32_t run,
                                          const ScanClear &clr) {
  int32_t o[kScanPer];
#pragma unroll
  for (int q = 0; q < kScanPer; ++q) {
    o[q] = run;
    run += v[q];
  }
  if (base + kScanPer <= n) {
#pragma unroll
    for (int q = 0; q < kScanPer / 4; ++q) {
      reinterpret_cast<int4 *>(out + base)[q] =
          make_int4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
      if (clr.counts) reinterpret_cast<int4 *>(clr.counts + base)[q] = make_int4(0, 0, 0, 0);
      if (clr.words) reinterpret_cast<int4 *>(clr.words + base)[q] = make_int4(0, 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kScanPer; ++q)
      if (base + q < n) {
        out[base + q] = o[q];
        if (clr.counts) clr.counts[base + q] = 0;
        if (clr.words) clr.words[base + q] = 0u;
      }
  }
}

// The whole scan by one workgroup of NT threads, NT x kScanPer elements at a
// time (every thread must call it; lds: NT / 64 entries).
template <int NT>
__device__ __forceinline__ void scan_by_block(const int32_t *in, int64_t n, int32_t *out,
                                              int32_t *lds, const ScanClear &clr) {
  int32_t before = 0;
  for (int64_t c = 0; c < n; c += (int64_t)NT * kScanPer) {
    const int64_t base = c + (int64_t)threadIdx.x * kScanPer;
    int32_t v[kScanPer];
    load_run(in, base, n, v);
    int32_t s = 0;
#pragma unroll
    for (int q = 0; q < kScanPer; ++q) s += v[q];
    int32_t total;
    const int32_t run = block_exclusive_scan<NT / 64>(s, lds, &total) + before;
    store_run(out, base, n, v, run, clr);
    before += total;
  }
  if (threadIdx.x == 0) out[n] = before;
}

// Atomic slots give an arbitrary order inside a cell; sort each cell's
// entries by (x key, caller index) so the layout (and every FP sum) is
// reproducible and each cell's particles are in x order.  Cells of at most
// kSmallCell entries are ranked one thread per particle (k_cell_rank);
// larger cells go to a list that whole workgroups sort (sort_big_cells).
constexpr int kSmallCell = 32;
constexpr int kSortChunk = 4096;  // entries a workgroup sorts at once in LDS
constexpr int kBigSortBlocks = 256;

// Order of two particles of one cell: by x key, then by caller index (the
// keys are x positions quantised to 2^-20 of the cell, so a cell's particles
// end up in x order and every extended row is x-sorted).
__device__ __forceinline__ uint64_t sort_key(const uint32_t *__restrict__ xq, int i) {
  return ((uint64_t)xq[i] << 32) | (uint32_t)i;
}

// A cell's sub-cell word from the x keys of its slots [a, b): nibble k
// (k = 0..6) counts its particles with x keys below (k + 1)/8 of the cell --
// with the particles in key order, the first slot of sub-cell k + 1 is the
// cell's first plus that count -- and nibble 7 counts them all; 0 (no
// sub-cells) for a cell of more than 15.  A nibble histogram of the
// sub-cells times 0x11111111 is its prefix sums.
__device__ __forceinline__ uint32_t sub_word(const uint32_t *__restrict__ skey, int a, int b) {
  if (b - a > 15) return 0u;
  uint32_t hist = 0;
  for (int p = a; p < b; ++p) hist += 1u << (4 * (skey[p] >> (20 - kXSubLog)));
  return hist * 0x11111111u;
}

// The sorted record of particle i: (x, y, z) wrapped into the box (0 when
// not finite) and rc clamped to [0, rc_cap] (NaN -> 0).
__device__ __forceinline__ double4 gather_record(const double L[3], double rc_cap, double px,
                                                 double py, double pz, double r) {
  double4 o;
  if (finite3(px, py, pz)) {
    o.x = wrap_coord(px, L[0]);
    o.y = wrap_coord(py, L[1]);
    o.z = wrap_coord(pz, L[2]);
  } else {
    o.x = o.y = o.z = 0.0;
  }
  o.w = (r >= 0.0) ? (r < rc_cap ? r : rc_cap) : 0.0;
  return o;
}

__device__ __forceinline__ double4 gather_record(const GatherOut &go, int i) {
  return gather_record(go.L, go.rc_cap, go.x[i], go.y[i], go.z[i], go.rc ? go.rc[i] : 0.0);
}

// Slot p of the cell-scattered order perm (x keys skey), in a cell of slots
// [a, b): the rank of its particle i there, the count of the cell's particles
// with smaller (x key, id).
__device__ __forceinline__ int rank_in_cell(const int32_t *__restrict__ perm,
                                            const uint32_t *__restrict__ skey, int64_t p, int i,
                                            int a, int b) {
  const uint32_t ki = skey[p];
  int r = 0;
  // four keys per round, all read before they are compared
  for (int q0 = a; q0 < b; q0 += 4) {
    uint32_t kj[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) kj[u] = q0 + u < b ? skey[q0 + u] : 0xffffffffu;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (q0 + u >= b) continue;
      r += kj[u] < ki ? 1 : 0;
      if (kj[u] == ki) r += perm[q0 + u] < i ? 1 : 0;  // equal keys (rare): by id
    }
  }
  return r;
}

// Per extended row (k_cells.hip, "periodic ghost images"): its particle count
// and F(-h_x), from the cell starts of its system.
__device__ __forceinline__ int32_t ext_row_count(const int32_t *__restrict__ cell_start,
                                                 const ExtGeom &g, int row, int32_t &row_lo) {
  const ExtRow r = ext_row(g, row);
  const int64_t T = cell_start[r.r0 + g.nc[0]] - cell_start[r.r0];
  const int64_t lo = row_prefix(cell_start, r.r0, g.nc[0], T, -g.h[0]);
  const int64_t hi = row_prefix(cell_start, r.r0, g.nc[0], T, g.nc[0] + g.h[0]);
  row_lo = (int32_t)lo;
  return (int32_t)(hi - lo);
}

// Up to this many extended rows one workgroup scans beside the rank (at 256
// threads about 1.5 us per 4096 rows; the rank of a system with so many rows
// takes longer).
constexpr int64_t kRowScanMax = 64 * 1024;

// One workgroup per listed cell: chunks of kSortChunk entries are sorted in
// LDS (bitonic), then runs are merged pairwise, each entry moving to its own
// offset in its run plus the count of smaller keys in the partner run (keys
// are distinct: they end in the caller index), ping-ponging between perm and
// tmp.  Entries are caller indices; their keys are looked up (sort_key).
// record(slot, id) writes the sorted record of particle id.
template <typename F>
__device__ __forceinline__ void sort_big_cells(const int32_t *__restrict__ cell_start,
                                               int32_t *perm, int32_t *tmp,
                                               const uint32_t *__restrict__ xq,
                                               const int32_t *__restrict__ big_list,
                                               const uint32_t *big_count, unsigned block,
                                               unsigned blocks, F &&record) {
  const int tid = threadIdx.x;
  const uint32_t nbig = *big_count;
  if (block >= nbig) return;
  __shared__ int32_t buf[kSortChunk];
  for (uint32_t q = block; q < nbig; q += blocks) {
    const int64_t c = big_list[q];
    const int a = cell_start[c], n = cell_start[c + 1] - a;
    for (int c0 = 0; c0 < n; c0 += kSortChunk) {
      const int len = n - c0 < kSortChunk ? n - c0 : kSortChunk;
      int P = 1;
      while (P < len) P <<= 1;
      // padding entries (-1) sort after every particle
      for (int i = tid; i < P; i += 256) buf[i] = i < len ? perm[a + c0 + i] : -1;
      __syncthreads();
      auto key = [&](int v) -> uint64_t { return v < 0 ? ~uint64_t(0) : sort_key(xq, v); };
      for (int k = 2; k <= P; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
          for (int i = tid; i < P; i += 256) {
            const int l = i ^ j;
            if (l > i) {
              const int u = buf[i], w = buf[l];
              if ((key(u) > key(w)) == ((i & k) == 0)) {
                buf[i] = w;
                buf[l] = u;
              }
            }
          }
          __syncthreads();
        }
      for (int i = tid; i < len; i += 256) perm[a + c0 + i] = buf[i];
      __syncthreads();
    }
    int32_t *src = perm + a, *dst = tmp + a;
    for (int L = kSortChunk; L < n; L <<= 1) {
      for (int p = tid; p < n; p += 256) {
        const int r = p / L, off = p - r * L;
        const int x = src[p];
        const uint64_t kx = sort_key(xq, x);
        const int o = (r ^ 1) * L;  // partner run
        int lo = 0, hi = 0;
        if (o < n) {
          hi = n - o < L ? n - o : L;
          while (lo < hi) {  // count of partner keys below x's
            const int m = (lo + hi) >> 1;
            if (sort_key(xq, src[o + m]) < kx) lo = m + 1;
            else hi = m;
          }
        }
        dst[(r & ~1) * L + off + lo] = x;
      }
      __syncthreads();
      int32_t *t = src;
      src = dst;
      dst = t;
    }
    if (src != perm + a) {
      for (int p = tid; p < n; p += 256) perm[a + p] = src[p];
      __syncthreads();
    }
    for (int p = tid; p < n; p += 256) record(c, a + p, perm[a + p]);
    __syncthreads();  // buf is free again
  }
}

}  // namespace dcm
