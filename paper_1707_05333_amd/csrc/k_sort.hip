// Grid hash and counting sort of the mesh-generating points, plus the
// prefix-sum and fill kernels the rest of the path uses.
//
// The sort realises the neighbour search the paper leaves to a tree
// (Sec. 3, the fast nearest-neighbour search): points are binned into a
// periodic grid of buckets, bucket-major with x fastest, so that the
// candidate stencil of a cell reads contiguous runs of positions.  Inside a
// bucket points keep their caller order, which makes the internal order, and
// every result downstream of it, independent of atomic scheduling.
#include <algorithm>

#include "mm_internal.h"

namespace mm {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ inline unsigned long long wave_incl_scan(unsigned long long x) {
  const int lane = __lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// Exclusive scan of one value per thread over a 256-thread block.
__device__ unsigned long long block_excl_scan(unsigned long long x, unsigned long long* total) {
  __shared__ unsigned long long wsum[kScanThreads / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const unsigned long long inc = wave_incl_scan(x);
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  unsigned long long base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kScanThreads / 64; ++k) {
    if (k < wid) base += wsum[k];
    tot += wsum[k];
  }
  __syncthreads();
  *total = tot;
  return base + inc - x;
}

// One block: sum of its tile.
template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const T* __restrict__ in, int64_t n,
                                                              unsigned long long* __restrict__ part) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k * kScanThreads + threadIdx.x;
    if (i < n) s += in[i];
  }
  unsigned long long tot;
  block_excl_scan(s, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Exclusive scan of the per-tile sums in place, by one block.
__global__ __launch_bounds__(kScanThreads) void k_scan_top(unsigned long long* part, int64_t m) {
  unsigned long long carry = 0;
  for (int64_t base = 0; base < m; base += kScanTile) {
    unsigned long long v[kScanItems];
    unsigned long long s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
      v[k] = (i < m) ? part[i] : 0ull;
      s += v[k];
    }
    unsigned long long tot;
    unsigned long long run = carry + block_excl_scan(s, &tot);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
      if (i < m) part[i] = run;
      run += v[k];
    }
    carry += tot;
    __syncthreads();
  }
}

// Sum of the tiles before this one: read from the scanned partials (top), or
// added up here from the raw ones (few tiles: cheaper than another launch).
__device__ unsigned long long tile_base(const unsigned long long* __restrict__ part, bool top) {
  if (top) return part[blockIdx.x];
  unsigned long long s = 0;
  for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kScanThreads) s += part[i];
  unsigned long long tot;
  block_excl_scan(s, &tot);
  return tot;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const T* __restrict__ in, int64_t n,
                                                            const unsigned long long* __restrict__ part, bool top,
                                                            unsigned long long* __restrict__ out) {
  __shared__ unsigned long long tile[kScanTile];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k * kScanThreads + threadIdx.x;
    tile[k * kScanThreads + threadIdx.x] = (i < n) ? in[i] : 0ull;
  }
  const unsigned long long before = tile_base(part, top);
  __syncthreads();
  unsigned long long v[kScanItems];
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = tile[threadIdx.x * kScanItems + k];
    s += v[k];
  }
  unsigned long long tot;
  unsigned long long run = before + block_excl_scan(s, &tot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    tile[threadIdx.x * kScanItems + k] = run;
    run += v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k * kScanThreads + threadIdx.x;
    if (i < n) out[i] = tile[k * kScanThreads + threadIdx.x];
  }
  // The last tile also writes the grand total at out[n].
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kScanThreads - 1) out[n] = run;
}

// Offsets of the assembled mesh from the packed face counts of the cells
// (faces << 32 | owned faces): off, the exclusive prefix sum of the counts,
// and soff, that of the slice widths (64 times the longest list of each 64
// consecutive cells).  A wavefront reads one slice per load, so a slice's
// width is a maximum over the wavefront.  The reduce pass sums both per tile;
// the down pass writes both, and the totals to the status block.
constexpr int kTileSlices = kScanTile / 64;

__device__ inline unsigned slice_width(unsigned long long c) {
  unsigned w = (unsigned)(c >> 32);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) w = max(w, (unsigned)__shfl_xor((int)w, o, 64));
  return 64u * w;
}

__global__ __launch_bounds__(kScanThreads) void k_mesh_reduce(const unsigned long long* __restrict__ counts, int64_t n,
                                                              unsigned long long* __restrict__ part,
                                                              unsigned long long* __restrict__ spart) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  unsigned long long s = 0, w = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k * kScanThreads + threadIdx.x;
    const unsigned long long c = i < n ? counts[i] : 0ull;
    s += c;
    const unsigned sl = slice_width(c);
    if ((threadIdx.x & 63) == 0) w += sl;
  }
  unsigned long long tot;
  block_excl_scan(s, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
  block_excl_scan(w, &tot);
  if (threadIdx.x == 0) spart[blockIdx.x] = tot;
}

// One tile of the down pass: its cells' offsets from `before`, its slices'
// from `sbefore`; returns the tile's sums.
__device__ void mesh_down_tile(const unsigned long long* __restrict__ counts, int64_t n, int64_t base,
                               unsigned long long before, unsigned long long sbefore,
                               unsigned long long* __restrict__ off, unsigned long long* __restrict__ soff,
                               unsigned long long* tile, unsigned* widths, unsigned long long* tot,
                               unsigned long long* stot) {
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int q = k * kScanThreads + threadIdx.x;
    const unsigned long long c = base + q < n ? counts[base + q] : 0ull;
    tile[q] = c;
    const unsigned sl = slice_width(c);
    if ((threadIdx.x & 63) == 0) widths[q >> 6] = sl;
  }
  __syncthreads();
  unsigned long long v[kScanItems];
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = tile[threadIdx.x * kScanItems + k];
    s += v[k];
  }
  unsigned long long run = before + block_excl_scan(s, tot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    tile[threadIdx.x * kScanItems + k] = run;
    run += v[k];
  }
  const unsigned long long sw = threadIdx.x < kTileSlices ? widths[threadIdx.x] : 0ull;
  const unsigned long long srun = sbefore + block_excl_scan(sw, stot);
  const int64_t slice = base / 64 + threadIdx.x;
  if (threadIdx.x < kTileSlices && 64 * slice < n) soff[slice] = srun;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int q = k * kScanThreads + threadIdx.x;
    if (base + q < n) off[base + q] = tile[q];
  }
}

__device__ void mesh_totals(unsigned long long total, unsigned long long stotal, int64_t n,
                            unsigned long long* off, unsigned long long* soff, DevStatus* st) {
  off[n] = total;
  soff[(n + 63) / 64] = stotal;
  st->n_faces = total & 0xffffffffull;
  st->n_csr = total >> 32;
}

__global__ __launch_bounds__(kScanThreads) void k_mesh_down(const unsigned long long* __restrict__ counts, int64_t n,
                                                            const unsigned long long* __restrict__ part,
                                                            const unsigned long long* __restrict__ spart, bool top,
                                                            unsigned long long* __restrict__ off,
                                                            unsigned long long* __restrict__ soff, DevStatus* st) {
  __shared__ unsigned long long tile[kScanTile];
  __shared__ unsigned widths[kTileSlices];
  const unsigned long long before = tile_base(part, top), sbefore = tile_base(spart, top);
  unsigned long long tot, stot;
  mesh_down_tile(counts, n, (int64_t)blockIdx.x * kScanTile, before, sbefore, off, soff, tile, widths, &tot, &stot);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) mesh_totals(before + tot, sbefore + stot, n, off, soff, st);
}

// Both passes in one block, for small meshes.
__global__ __launch_bounds__(kScanThreads) void k_mesh_scan_small(const unsigned long long* __restrict__ counts,
                                                                  int64_t n, unsigned long long* __restrict__ off,
                                                                  unsigned long long* __restrict__ soff,
                                                                  DevStatus* st) {
  __shared__ unsigned long long tile[kScanTile];
  __shared__ unsigned widths[kTileSlices];
  unsigned long long before = 0, sbefore = 0;
  for (int64_t base = 0; base < n; base += kScanTile) {
    unsigned long long tot, stot;
    mesh_down_tile(counts, n, base, before, sbefore, off, soff, tile, widths, &tot, &stot);
    before += tot;
    sbefore += stot;
    __syncthreads();
  }
  if (threadIdx.x == 0) mesh_totals(before, sbefore, n, off, soff, st);
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Status of a launch set: everything (a new call), or, before the second
// tessellation of a step, the counters of the mesh only.
__device__ void reset_status(DevStatus* s, SegStatus* segst, int nseg, bool remesh) {
  const int t = threadIdx.x;
  if (t == 0) {
    s->n_deferred = 0;
    s->n_overflow = 0;
    s->n_dense = 0;
    s->n_dense_cells = 0;
    s->n_redo = 0;
    s->n_dredo = 0;
    s->n_sub = 0;
    s->n_faces = 0;
    s->n_csr = 0;
    if (!remesh) {
      s->flags = 0;
      s->max_faces = 0;
      s->bad_cell = 0x7fffffff;
      s->asym_cell = -1;
      s->asym_nbr = -1;
    }
  }
  if (remesh) return;
  for (int k = t; k < nseg; k += blockDim.x) {
    SegStatus& g = segst[k];
    g.dt_bits = 0x7ff0000000000000ull;   // +inf
    g.flags = 0;
    g.bad_cell = 0x7fffffff;
    for (int q = 0; q < 4; ++q) g.floor_hits[q] = 0;
  }
}

__global__ void k_status_reset(DevStatus* s, SegStatus* segst, int nseg) { reset_status(s, segst, nseg, false); }

// Start of a tessellation: block 0 resets the status; every block clears its
// part of the bucket counters and, with host_segs set, copies its part of the
// segment table from pinned host memory (one segment: the descriptor travels as
// an argument, `one`).  One block's loads from the host are too few in flight for
// a large table: with it and one block publishing the reports, a step of 16,384
// simulations of 64 points took 8.0 ms instead of 5.5, and one of 4,096 2.04
// instead of 1.48.
__global__ __launch_bounds__(256) void k_begin(SegDesc one, const SegDesc* __restrict__ host_segs, SegDesc* segs,
                                               int nseg, bool remesh, uint32_t* __restrict__ bcount, int64_t nbt,
                                               DevStatus* st, SegStatus* segst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nbt) bcount[i] = 0u;
  if (host_segs && !remesh) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(host_segs);
    uint64_t* dst = reinterpret_cast<uint64_t*>(segs);
    for (int64_t k = i; k < (int64_t)(sizeof(SegDesc) / 8) * nseg; k += (int64_t)gridDim.x * blockDim.x) dst[k] = src[k];
  }
  if (blockIdx.x != 0) return;
  reset_status(st, segst, nseg, remesh);
  if (!host_segs && !remesh && threadIdx.x == 0) segs[0] = one;
}

// Copies the status of the launch set and of its segments to pinned host
// memory (visible to the host once the stream has been waited for).
__global__ __launch_bounds__(256) void k_publish(const DevStatus* __restrict__ st, const SegStatus* __restrict__ segst,
                                                 int nseg, DevStatus* host_st, SegStatus* host_segst) {
  static_assert(sizeof(DevStatus) % 8 == 0 && sizeof(SegStatus) % 8 == 0, "copied in 8-byte words");
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t* a = reinterpret_cast<const uint64_t*>(st);
  uint64_t* b = reinterpret_cast<uint64_t*>(host_st);
  if (t < (int64_t)(sizeof(DevStatus) / 8)) b[t] = a[t];
  const uint64_t* c = reinterpret_cast<const uint64_t*>(segst);
  uint64_t* d = reinterpret_cast<uint64_t*>(host_segst);
  for (int64_t k = t; k < (int64_t)(sizeof(SegStatus) / 8) * nseg; k += (int64_t)gridDim.x * blockDim.x) d[k] = c[k];
}

// Bucket of a point in its segment's grid, or the grid's first bucket for a
// position that is not finite or outside [0, L) (the caller fails the call).
__device__ inline int64_t point_bucket(const GridParams& g, double x, double y, double z, bool* ok) {
  *ok = (x >= 0.0) && (x < g.L[0]) && (y >= 0.0) && (y < g.L[1]) && (z >= 0.0) && (z < g.L[2]);
  if (!*ok) return g.base;
  return g.base + bucket_key(g.nb, bucket_coord(x, g.inv_hb[0], g.nb[0]), bucket_coord(y, g.inv_hb[1], g.nb[1]),
                             bucket_coord(z, g.inv_hb[2], g.nb[2]));
}

// Bucket key of every used slot (the segment's first bucket plus the bucket
// of the point in that segment's grid; -1 for an unused slot), and the
// point's arrival rank in its bucket.
__global__ void k_hash(const double* __restrict__ pos, int64_t n_slots, const int32_t* __restrict__ slot_seg,
                       const SegDesc* __restrict__ segs, int32_t* __restrict__ key, int32_t* __restrict__ rank,
                       uint32_t* bcount, DevStatus* st, SegStatus* segst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_slots) return;
  const int seg = slot_seg ? slot_seg[i] : 0;
  if (seg < 0) {
    key[i] = -1;
    return;
  }
  bool ok;
  const int64_t k = point_bucket(segs[seg].g, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], &ok);
  if (!ok) seg_fail(st, segst, seg, F_BADPOS, (int)i);
  key[i] = (int32_t)k;
  rank[i] = (int32_t)atomicAdd(&bcount[k], 1u);
}

__global__ void k_scatter(const int32_t* __restrict__ key, const int32_t* __restrict__ rank, int64_t n_slots,
                          const unsigned long long* __restrict__ boff, int32_t* __restrict__ perm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_slots) return;
  const int k = key[i];
  if (k >= 0) perm[boff[k] + (unsigned)rank[i]] = (int32_t)i;
}

// Internal cell s holds slot q.
__device__ inline void put_cell(int64_t s, int32_t q, const double* __restrict__ pos,
                                const int32_t* __restrict__ slot_seg, int32_t* __restrict__ perm,
                                double* __restrict__ spos, int32_t* __restrict__ sseg) {
  perm[s] = q;
  sseg[s] = slot_seg ? slot_seg[q] : 0;
  const double* p = pos + 3 * (int64_t)q;
  const double x = p[0], y = p[1], z = p[2];
  spos[3 * s] = x;
  spos[3 * s + 1] = y;
  spos[3 * s + 2] = z;
}

// A bucket of more than kDense points: takes room for its sub-offset table
// (s^3 + 1 entries; which room does not matter), joins the list the block
// sort takes, and lists its cells (sorted positions) for the tessellation's
// dense passes.
__device__ inline void list_dense(int64_t b, int64_t lo, int cnt, unsigned long long* __restrict__ sbase,
                                  int32_t* __restrict__ dense, int32_t* __restrict__ dcells, DevStatus* st) {
  const int s = sub_size((unsigned)cnt);
  sbase[b] = (unsigned long long)atomicAdd(&st->n_sub, s * s * s + 1);
  dense[atomicAdd(&st->n_dense, 1)] = (int32_t)b;
  const int c0 = atomicAdd(&st->n_dense_cells, cnt);
  for (int i = 0; i < cnt; ++i) dcells[c0 + i] = (int32_t)(lo + i);
}

// Per bucket: a bucket of at most kDense points gets its slot order back
// (ranks by counting, in registers: the scatter filled it in arrival order)
// and its cells' positions; a denser one is listed for the block sort, which
// does both.  Buckets above kDenseMax points fail the call: their points stay
// where the scatter put them and are read whole.  They are listed in pieces of
// kDenseMax cells (the last one ends with the bucket, over the one before), as
// -1 - first cell, for the block sort to write positions and segments: a blown-up
// state may have every point in one bucket, and this thread alone took 66 ms for
// 262,144 of them.
__global__ void k_bucket_prep(const unsigned long long* __restrict__ boff, int64_t nbt, const double* __restrict__ pos,
                              const int32_t* __restrict__ slot_seg, int32_t* perm, double* __restrict__ spos,
                              int32_t* __restrict__ sseg, unsigned long long* __restrict__ sbase,
                              int32_t* __restrict__ dense, int32_t* __restrict__ dcells, DevStatus* st,
                              SegStatus* segst) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbt) return;
  const int64_t lo = (int64_t)boff[b];
  const int64_t cnt = (int64_t)boff[b + 1] - lo;
  if (cnt <= kDense) {
    int32_t v[kDense];
#pragma unroll
    for (int k = 0; k < kDense; ++k) v[k] = k < cnt ? perm[lo + k] : 0x7fffffff;
#pragma unroll
    for (int k = 0; k < kDense; ++k) {
      if (k < cnt) {
        int r = 0;
#pragma unroll
        for (int m = 0; m < kDense; ++m) r += v[m] < v[k];
        put_cell(lo + r, v[k], pos, slot_seg, perm, spos, sseg);
      }
    }
    return;
  }
  if (cnt > kDenseMax) {
    seg_fail(st, segst, slot_seg ? slot_seg[perm[lo]] : 0, F_DENSE, (int)lo);
    const int pieces = (int)((cnt + kDenseMax - 1) / kDenseMax);
    const int d0 = atomicAdd(&st->n_dense, pieces);
    for (int k = 0; k < pieces; ++k)
      dense[d0 + k] = (int32_t)(-1 - (k + 1 < pieces ? lo + (int64_t)k * kDenseMax : lo + cnt - kDenseMax));
    return;
  }
  list_dense(b, lo, (int)cnt, sbase, dense, dcells, st);
}

// The whole counting sort of one small segment in one block (status,
// segment descriptor and bucket counts included), its counts and order in
// LDS: a dozen launches of a few microseconds each become one.  Dense
// buckets are left to the block sort, as above.
constexpr int kSmallThreads = 1024;
constexpr int kSmallItems = 8;
constexpr int kSmallPoints = kSmallThreads * kSmallItems;
constexpr int kSmallBuckets = kSmallPoints + 8;

__global__ __launch_bounds__(kSmallThreads) void k_sort_small(SegDesc one, SegDesc* segs, bool remesh,
                                                              const double* __restrict__ pos, int n,
                                                              unsigned long long* __restrict__ boff,
                                                              unsigned long long* __restrict__ sbase,
                                                              int32_t* __restrict__ dense, int32_t* __restrict__ perm,
                                                              int32_t* __restrict__ sseg, double* __restrict__ spos,
                                                              int32_t* __restrict__ dcells, DevStatus* st,
                                                              SegStatus* segst) {
  __shared__ uint32_t cnt[kSmallBuckets];   // bucket counts, then first positions
  __shared__ int32_t order[kSmallPoints];
  __shared__ uint32_t wsum[kSmallThreads / 64];
  const int t = threadIdx.x;
  const GridParams& g = one.g;
  const int nbt = g.nbt;
  for (int b = t; b < nbt; b += kSmallThreads) cnt[b] = 0u;
  reset_status(st, segst, 1, remesh);
  if (t == 0 && !remesh) segs[0] = one;
  __syncthreads();
  int key[kSmallItems], rank[kSmallItems];
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k) {
    const int i = t + k * kSmallThreads;
    key[k] = -1;
    if (i < n) {
      bool ok;
      key[k] = (int)point_bucket(g, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], &ok);
      if (!ok) seg_fail(st, segst, 0, F_BADPOS, i);
      rank[k] = (int)atomicAdd(&cnt[key[k]], 1u);
    }
  }
  __syncthreads();
  // Exclusive scan of the counts, one contiguous run of buckets per thread.
  const int per = (nbt + kSmallThreads - 1) / kSmallThreads;
  const int b0 = min(t * per, nbt), b1 = min(b0 + per, nbt);
  uint32_t sum = 0;
  for (int b = b0; b < b1; ++b) sum += cnt[b];
  const uint32_t incl = (uint32_t)wave_incl_scan(sum);
  if ((t & 63) == 63) wsum[t >> 6] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int k = 0; k < (t >> 6); ++k) run += wsum[k];
  for (int b = b0; b < b1; ++b) {
    const uint32_t c = cnt[b];
    cnt[b] = run;
    run += c;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSmallItems; ++k)
    if (key[k] >= 0) order[cnt[key[k]] + rank[k]] = t + k * kSmallThreads;
  for (int b = t; b < nbt; b += kSmallThreads) boff[b] = cnt[b];
  if (t == 0) boff[nbt] = (unsigned long long)n;
  __syncthreads();
  for (int b = t; b < nbt; b += kSmallThreads) {
    const int lo = (int)cnt[b], c = (b + 1 < nbt ? (int)cnt[b + 1] : n) - lo;
    if (c > kDenseMax) {
      seg_fail(st, segst, 0, F_DENSE, lo);
    } else if (c > kDense) {
      list_dense(b, lo, c, sbase, dense, dcells, st);
    } else {
      for (int a = 1; a < c; ++a) {   // slot order of a handful
        const int32_t v = order[lo + a];
        int m = a - 1;
        while (m >= 0 && order[lo + m] > v) {
          order[lo + m + 1] = order[lo + m];
          --m;
        }
        order[lo + m + 1] = v;
      }
    }
  }
  __syncthreads();
  for (int s = t; s < n; s += kSmallThreads) put_cell(s, order[s], pos, nullptr, perm, spos, sseg);
}

// Orders the points of each dense bucket by sub-bucket (x fastest), then by
// slot, with a bitonic sort of (sub-bucket << 32 | slot) keys in LDS, and
// writes the bucket's sub-bucket offsets: entry k counts its points in
// sub-buckets below k (k = 0 .. s^3).  One block per entry of the list.
constexpr int kDenseThreads = 256;

__global__ __launch_bounds__(kDenseThreads) void k_dense_order(
    const int32_t* __restrict__ dense, const DevStatus* __restrict__ st, const unsigned long long* __restrict__ boff,
    const unsigned long long* __restrict__ sbase, const double* __restrict__ pos,
    const int32_t* __restrict__ slot_seg, const SegDesc* __restrict__ segs, int32_t* __restrict__ perm,
    double* __restrict__ spos, int32_t* __restrict__ sseg, uint32_t* __restrict__ soffs) {
  __shared__ unsigned long long kv[kDenseMax];
  const int nd = st->n_dense;
  const int t = threadIdx.x;
  for (int it = blockIdx.x; it < nd; it += gridDim.x) {
    const int64_t b = dense[it];
    if (b < 0) {   // a piece of a bucket beyond the sort
      for (int64_t s = -1 - b + t; s < -1 - b + kDenseMax; s += kDenseThreads)
        put_cell(s, perm[s], pos, slot_seg, perm, spos, sseg);
      continue;
    }
    const int64_t lo = (int64_t)boff[b];
    const int cnt = (int)((int64_t)boff[b + 1] - lo);
    const int s = sub_size((unsigned)cnt);
    int p2 = 1;
    while (p2 < cnt) p2 <<= 1;
    const int seg = slot_seg ? slot_seg[perm[lo]] : 0;
    const GridParams& g = segs[seg].g;
    for (int i = t; i < p2; i += kDenseThreads) {
      unsigned long long k = ~0ull;
      if (i < cnt) {
        const int32_t q = perm[lo + i];
        int sc[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double x = pos[3 * (int64_t)q + a];
          sc[a] = sub_coord(x, g.inv_hb[a], bucket_coord(x, g.inv_hb[a], g.nb[a]), s);
        }
        k = ((unsigned long long)((sc[2] * s + sc[1]) * s + sc[0]) << 32) | (uint32_t)q;
      }
      kv[i] = k;
    }
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = t; i < p2; i += kDenseThreads) {
          const int ixj = i ^ j;
          if (ixj > i) {
            const unsigned long long a = kv[i], c = kv[ixj];
            if (((i & k) == 0) == (a > c)) {
              kv[i] = c;
              kv[ixj] = a;
            }
          }
        }
        __syncthreads();
      }
    }
    for (int i = t; i < cnt; i += kDenseThreads)
      put_cell(lo + i, (int32_t)(uint32_t)(kv[i] & 0xffffffffull), pos, slot_seg, perm, spos, sseg);
    const int ns = s * s * s;
    uint32_t* so = soffs + sbase[b];
    for (int k = t; k <= ns; k += kDenseThreads) {
      // first position whose sub-bucket is k or more
      const unsigned long long key = (unsigned long long)k << 32;
      int l = 0, h = cnt;
      while (l < h) {
        const int m = (l + h) >> 1;
        if (kv[m] < key) l = m + 1;
        else h = m;
      }
      so[k] = (uint32_t)l;
    }
    __syncthreads();
  }
}

inline unsigned blocks_for(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

// Tiles up to which each block of a down pass adds up the tiles before it by
// itself (a few KB from L2) instead of a launch that scans them first.
constexpr int64_t kOwnBaseTiles = 2048;

size_t scan_tmp_elems(int64_t n) { return 2 * ((size_t)((n + kScanTile - 1) / kScanTile) + 1); }

void launch_mesh_scan(const unsigned long long* counts, int64_t n, unsigned long long* off, unsigned long long* soff,
                      unsigned long long* tmp, DevStatus* st_dev, hipStream_t st) {
  // One block takes about 2 us per tile, a launch about 4.5 us.
  if (n <= 2 * kScanTile) {
    hipLaunchKernelGGL(k_mesh_scan_small, dim3(1), dim3(kScanThreads), 0, st, counts, n, off, soff, st_dev);
    return;
  }
  const int64_t tiles = (n + kScanTile - 1) / kScanTile;
  const bool top = tiles > kOwnBaseTiles;
  unsigned long long* stmp = tmp + tiles;
  hipLaunchKernelGGL(k_mesh_reduce, dim3((unsigned)tiles), dim3(kScanThreads), 0, st, counts, n, tmp, stmp);
  if (top) {
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanThreads), 0, st, tmp, tiles);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanThreads), 0, st, stmp, tiles);
  }
  hipLaunchKernelGGL(k_mesh_down, dim3((unsigned)tiles), dim3(kScanThreads), 0, st, counts, n, tmp, stmp, top, off,
                     soff, st_dev);
}

void launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(n, 256)), dim3(256), 0, st, p, v, n);
}

void launch_status_reset(DevStatus* s, SegStatus* segst, int nseg, hipStream_t st) {
  hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(256), 0, st, s, segst, nseg);
}

void launch_publish(const DevStatus* s, const SegStatus* segst, int nseg, DevStatus* host_s, SegStatus* host_segst,
                    hipStream_t st) {
  const int64_t words = (int64_t)(sizeof(SegStatus) / 8) * nseg;
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>((words + 255) / 256, 1024));
  hipLaunchKernelGGL(k_publish, dim3(blocks), dim3(256), 0, st, s, segst, nseg, host_s, host_segst);
}

void launch_sort(const double* pos, int64_t n_slots, const int32_t* slot_seg, const SegDesc* segs_host, SegDesc* segs,
                 int nseg, bool remesh, int64_t nbt, uint32_t* bcount, unsigned long long* boff,
                 unsigned long long* scan_tmp, unsigned long long* sbase, uint32_t* soffs, int32_t* key, int32_t* rank,
                 int32_t* perm, int32_t* sseg, double* spos, int32_t* dcells, DevStatus* st_dev, SegStatus* segst,
                 hipStream_t st) {
  const bool one = nseg == 1;
  // One block sorts a small segment (about 1.5 us per 1,024 points, against
  // five more launches of about 4.5 us each).
  if (one && !slot_seg && n_slots <= kSmallPoints && nbt <= kSmallBuckets) {
    hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(kSmallThreads), 0, st, segs_host[0], segs, remesh, pos,
                       (int)n_slots, boff, sbase, key, perm, sseg, spos, dcells, st_dev, segst);
  } else {
    hipLaunchKernelGGL(k_begin, dim3(std::max(1u, blocks_for(nbt, 256))), dim3(256), 0, st,
                       one ? segs_host[0] : SegDesc{}, one ? nullptr : segs_host, segs, nseg, remesh, bcount, nbt,
                       st_dev, segst);
    hipLaunchKernelGGL(k_hash, dim3(blocks_for(n_slots, 256)), dim3(256), 0, st, pos, n_slots, slot_seg, segs, key,
                       rank, bcount, st_dev, segst);
    const int64_t tiles = (nbt + kScanTile - 1) / kScanTile;
    const bool top = tiles > kOwnBaseTiles;
    if (tiles > 1)
      hipLaunchKernelGGL(k_scan_reduce<uint32_t>, dim3((unsigned)tiles), dim3(kScanThreads), 0, st, bcount, nbt,
                         scan_tmp);
    if (top) hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanThreads), 0, st, scan_tmp, tiles);
    hipLaunchKernelGGL(k_scan_down<uint32_t>, dim3((unsigned)tiles), dim3(kScanThreads), 0, st, bcount, nbt, scan_tmp,
                       top, boff);
    hipLaunchKernelGGL(k_scatter, dim3(blocks_for(n_slots, 256)), dim3(256), 0, st, key, rank, n_slots, boff, perm);
    // key (read by the scatter) now takes the list of dense buckets.
    hipLaunchKernelGGL(k_bucket_prep, dim3(blocks_for(nbt, 256)), dim3(256), 0, st, boff, nbt, pos, slot_seg, perm,
                       spos, sseg, sbase, key, dcells, st_dev, segst);
  }
  const unsigned dense_blocks = (unsigned)std::min<int64_t>(std::max<int64_t>(nbt / kDense, 1), 2048);
  hipLaunchKernelGGL(k_dense_order, dim3(dense_blocks), dim3(kDenseThreads), 0, st, key, st_dev, boff, sbase, pos,
                     slot_seg, segs, perm, spos, sseg, soffs);
}

}  // namespace mm
