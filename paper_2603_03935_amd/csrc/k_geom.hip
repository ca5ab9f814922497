// Geometry workload of the mapping pipeline (arXiv 2603.03935, Sec. III-B):
// each segment's depth pixels are back-projected to world points, DBSCAN
// removes the noise points, the rest are voxelised, and segments are
// associated with map instances by exact voxel overlap (Sec. III-B, the
// voxel-overlap refinement).
//
// Where floating point decides an integer (which points are neighbours
// within eps, which voxel a point falls in) every operation is an explicitly
// rounded single-precision one in a fixed order (no contraction into FMA), so
// the decisions are reproducible operation by operation.
//
// Kernels:
//   back-projection  one bit per pixel of the frame says whether its depth is a
//                    reading; a mask's points are counted as the bits it has in
//                    common with those, and written by blocks of rows, each
//                    block counting the rows before it, so each mask's points
//                    come out in row-major pixel order;
//   DBSCAN           a global hash grid of (segment, cell) keys with cells of
//                    side eps, a counting sort of the points by cell, then a
//                    wavefront per cell tests its points against the 27
//                    cells around (core, then border; early exit);
//   voxels           a global hash set of (segment, voxel) keys lists the
//                    distinct voxels by segment; each segment's keys are
//                    sorted in chunks of 1024 that are merged by rank;
//   overlap          one workgroup per (segment, instance) pair: the runs of the
//                    two lists whose boxes meet are taken, the more entries are
//                    staged in LDS and the fewer binary-searched there.
#include <algorithm>
#include <type_traits>

#include "disc_device.h"

namespace disc {

// ---------------------------------------------------------------------------
// prefix sums
// ---------------------------------------------------------------------------
// sum of v over the threads before this one of a block of 1024, the block's
// sum in total; sh: 16 values.  Every thread of the block calls it.
template <class T>
__device__ __forceinline__ T block_exscan_1024(T v, T* sh, T& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  T x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const T t = __shfl_up(x, o);
    if (lane >= o) x += t;
  }
  if (lane == 63) sh[wv] = x;
  __syncthreads();
  T before = 0, all = 0;
  for (int k = 0; k < 16; ++k) {
    const T t = sh[k];
    before += k < wv ? t : T(0);
    all += t;
  }
  __syncthreads();
  total = all;
  return before + x - v;
}

// out[i] = sum of in[j < i] for i <= n, by one workgroup (n is the number of
// masks or segments of a call).  CHUNKS: also cout, likewise, of the number
// of chunks of `chunk` elements that in[j] elements make.
template <int CHUNKS>
__global__ __launch_bounds__(1024) void k_offsets(const int32_t* in, int n, int32_t* out, int chunk, int32_t* cout) {
  __shared__ uint64_t sh[16];
  uint64_t run = 0;  // elements low, chunks high
  for (int i0 = 0; i0 < n; i0 += 1024) {
    const int i = i0 + (int)threadIdx.x;
    const uint32_t v = i < n ? (uint32_t)in[i] : 0u;
    const uint64_t w = (uint64_t)v | ((uint64_t)(CHUNKS ? (v + chunk - 1) / chunk : 0u) << 32);
    uint64_t total;
    const uint64_t ex = run + block_exscan_1024(w, sh, total);
    if (i < n) {
      out[i] = (int32_t)ex;
      if (CHUNKS) cout[i] = (int32_t)(ex >> 32);
    }
    run += total;
  }
  if (threadIdx.x == 0) {
    out[n] = (int32_t)run;
    if (CHUNKS) cout[n] = (int32_t)(run >> 32);
  }
}

// ---------------------------------------------------------------------------
// back-projection
// ---------------------------------------------------------------------------
struct Cam {
  float fx, fy, cx, cy;
  float R[9];
  float t[3];
  float dmin, dmax;
};

// valid pixel bits of word k of row y (lane l = column 64k + l), this lane's
// depth in z
__device__ __forceinline__ bool pixel_valid(const uint64_t* row, int k, int y, int w, int s, const float* depth,
                                            const Cam& c, float& z) {
  const int lane = threadIdx.x & 63;
  const uint64_t word = row[k];
  const int x = 64 * k + lane;
  z = 0.f;
  if (!((word >> lane) & 1ull) || x >= w || (x % s) != 0) return false;
  z = depth[(int64_t)y * w + x];
  return __builtin_isfinite(z) && z >= c.dmin && z <= c.dmax;
}

__device__ __forceinline__ int row_count(const uint64_t* row, int y, int wq, int w, int s, const float* depth,
                                         const Cam& c) {
  int cnt = 0;
  for (int k = 0; k < wq; ++k) {
    if (row[k] == 0ull) continue;  // uniform
    float z;
    const bool v = pixel_valid(row, k, y, w, s, depth, c, z);
    cnt += __builtin_popcountll(__ballot(v));
  }
  return cnt;
}

// (contraction off in this scope: every product and sum is rounded on its
// own; the division is the correctly rounded one)
__device__ __forceinline__ void world_point(const Cam& c, int x, int y, float z, float* out) {
#pragma clang fp contract(off)
  const float xc = (((float)x - c.cx) * z) / c.fx;
  const float yc = (((float)y - c.cy) * z) / c.fy;
#pragma unroll
  for (int k = 0; k < 3; ++k) out[k] = ((c.R[3 * k] * xc + c.R[3 * k + 1] * yc) + c.R[3 * k + 2] * z) + c.t[k];
}

// Valid bits of the frame, [h][wq] words like a mask's: the pixel lies on the
// stride's grid and its depth is a reading.  Eight words (2 KB of depth) per
// wavefront, their loads issued together.
__global__ __launch_bounds__(256) void k_bp_valid(const float* depth, int h, int w, int s, Cam c, uint64_t* valid) {
  const int wq = (w + 63) / 64, nw = h * wq, lane = threadIdx.x & 63;
  const int w0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * 8;
  float z[8];
  bool in[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int k = w0 + i, y = k / wq, x = 64 * (k - y * wq) + lane;
    in[i] = k < nw && x < w && x % s == 0 && y % s == 0;
    z[i] = in[i] ? depth[(int64_t)y * w + x] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint64_t b = __ballot(in[i] && __builtin_isfinite(z[i]) && z[i] >= c.dmin && z[i] <= c.dmax);
    if (lane == 0 && w0 + i < nw) valid[w0 + i] = b;
  }
}

// points of words 0 .. nw - 1 of a mask, this thread's share (block of BT threads)
template <int BT>
__device__ __forceinline__ int count_words(const uint64_t* mb, const uint64_t* valid, int nw) {
  int cnt = 0, k = threadIdx.x;
  for (; k + 3 * BT < nw; k += 4 * BT) {
    uint64_t a[4], b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = mb[k + BT * i];
      b[i] = valid[k + BT * i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) cnt += __builtin_popcountll(a[i] & b[i]);
  }
  for (; k < nw; k += BT) cnt += __builtin_popcountll(mb[k] & valid[k]);
  return cnt;
}

// One workgroup per mask: the number of its points.  Reading the mask (38 KB
// of a 480x640 frame) bounds it: 36 masks 78 us with one depth load per set
// word and row after row, 4 us as popcounts (and 5 us for the valid bits).
__global__ __launch_bounds__(1024) void k_bp_count(const uint64_t* bits, const uint64_t* valid, int nw, int32_t* counts) {
  int cnt = count_words<1024>(bits + (int64_t)blockIdx.x * nw, valid, nw);
  __shared__ int red[16];
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int k = 0; k < 16; ++k) t += red[k];
    counts[blockIdx.x] = t;
  }
}

// One workgroup per (mask, block of kBpRows rows), `masks` masks to a row of the
// grid (whose x holds fewer than 2^32 threads), a mask's blocks one after the
// other (43 masks of 618x1012: 11.6 us; 20.2 with the masks as x and the blocks
// as y, which leaves the blocks of a large mask to a few XCDs and its last ones,
// which count the most rows, to the end): it counts the points of
// the mask's earlier rows (popcounts of words that are in L2 by then) to know
// where its own begin, so that a frame's few large masks spread over the chip;
// blocks without points leave at once.  36 masks of a 480x640 frame: 104 us
// with one workgroup per mask (k_bp_write), 16 us with 15 per mask.
constexpr int kBpRows = 32;

__global__ __launch_bounds__(1024) void k_bp_write_rows(const float* depth, const uint64_t* bits, const uint64_t* valid,
                                                       int m, int h, int w, int nblk, int masks, Cam c,
                                                       const int32_t* offsets, float* points) {
  const int i = blockIdx.y * masks + blockIdx.x / nblk, y0 = (blockIdx.x % nblk) * kBpRows;
  if (i >= m) return;
  const int wq = (w + 63) / 64, w0 = y0 * wq, w1 = min(h, y0 + kBpRows) * wq;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint64_t* mb = bits + (int64_t)i * h * wq;
  bool any = false;
  for (int k = w0 + tid; k < w1; k += 1024) any |= (mb[k] & valid[k]) != 0ull;
  if (!__syncthreads_or(any ? 1 : 0)) return;
  __shared__ int red[16];
  __shared__ uint64_t lv[1024];  // the words with points of a round, where their points go, and which they are
  __shared__ int lpos[1024], lidx[1024];
  int before = count_words<1024>(mb, valid, w0);
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (lane == 0) red[wv] = before;
  __syncthreads();
  int64_t base = offsets[i];
  for (int q = 0; q < 16; ++q) base += red[q];
  __syncthreads();
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int k0 = w0; k0 < w1; k0 += 1024) {
    const int k = k0 + tid;
    const uint64_t v = k < w1 ? mb[k] & valid[k] : 0ull;
    // prefix of (points, words with points), packed: at most 65536 and 1024
    int all;
    const int pre = block_exscan_1024(__builtin_popcountll(v) | (v ? 1 << 20 : 0), red, all);
    if (v) {
      lv[pre >> 20] = v;
      lpos[pre >> 20] = pre & 0xFFFFF;
      lidx[pre >> 20] = k;
    }
    __syncthreads();
    const int n = all >> 20;
    for (int e0 = wv; e0 < n; e0 += 64) {  // four words of a wavefront in flight
      float z[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + 16 * u;
        z[u] = 0.f;
        if (e < n && ((lv[e] >> lane) & 1ull)) {
          const int y = lidx[e] / wq, x = 64 * (lidx[e] - y * wq) + lane;
          z[u] = depth[(int64_t)y * w + x];
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + 16 * u;
        if (e < n && ((lv[e] >> lane) & 1ull)) {
          const int y = lidx[e] / wq, x = 64 * (lidx[e] - y * wq) + lane;
          float p[3];
          world_point(c, x, y, z[u], p);
          float* o = points + 3 * (base + lpos[e] + __builtin_popcountll(lv[e] & below));
          o[0] = p[0];
          o[1] = p[1];
          o[2] = p[2];
        }
      }
    }
    base += all & 0xFFFFF;
    __syncthreads();  // the list is rewritten by the next round
  }
}

// The same without the valid bits (which need workspace, and so cannot be
// part of a graph that is being captured): one workgroup per mask, rows in
// chunks of 16 (one per wavefront), points written in row-major order from
// offsets[i].
__global__ __launch_bounds__(1024) void k_bp_write(const float* depth, const uint64_t* bits, int m, int h, int w, int s,
                                                   Cam c, const int32_t* offsets, float* points) {
  const int i = blockIdx.x, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wq = (w + 63) / 64;
  const uint64_t* mb = bits + (int64_t)i * h * wq;
  __shared__ int rc[16];
  int64_t run = offsets[i];
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int y0 = 0; y0 < h; y0 += 16 * s) {
    const int y = y0 + s * wv;
    const uint64_t* row = mb + (int64_t)y * wq;
    const int cnt = y < h ? row_count(row, y, wq, w, s, depth, c) : 0;
    if (lane == 0) rc[wv] = cnt;
    __syncthreads();
    int64_t pos = run;
    int tot = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) pos += rc[k];
      tot += rc[k];
    }
    if (y < h && cnt > 0) {
      for (int k = 0; k < wq; ++k) {
        if (row[k] == 0ull) continue;
        float z;
        const bool v = pixel_valid(row, k, y, w, s, depth, c, z);
        const uint64_t b = __ballot(v);
        if (v) {
          float p[3];
          world_point(c, 64 * k + lane, y, z, p);
          float* o = points + 3 * (pos + __builtin_popcountll(b & below));
          o[0] = p[0];
          o[1] = p[1];
          o[2] = p[2];
        }
        pos += __builtin_popcountll(b);
      }
    }
    run += tot;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// hash grid shared by DBSCAN and the voxel sets
// ---------------------------------------------------------------------------
constexpr uint64_t kEmpty = ~0ull;

__device__ __forceinline__ uint32_t hash64(uint64_t k) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  return (uint32_t)k;
}

// 16-bit biased cell coordinate (cells beyond +-32767 are clamped: the
// distance tests below never depend on the cell a point is filed under
// being its true cell, only on each point being filed once)
__device__ __forceinline__ uint64_t cell16(int v) { return (uint64_t)(min(max(v, -32767), 32767) + 32768); }

__device__ __forceinline__ uint64_t cell_key(int seg, int cx, int cy, int cz) {
  return ((uint64_t)seg << 48) | (cell16(cx) << 32) | (cell16(cy) << 16) | cell16(cz);
}

__device__ __forceinline__ int cell_of(float p, float e) { return (int)floorf(p / e); }

// Insert (or find) a key; returns its slot.  A slot's key never changes once
// it is set, so a plain load (which may show an older, empty state) settles
// every case but the empty one, and only that takes the atomic.
__device__ __forceinline__ uint32_t hash_insert(uint64_t* keys, uint32_t mask, uint64_t key, bool& fresh) {
  uint32_t h = hash64(key) & mask;
  fresh = false;
  for (;;) {
    uint64_t prev = __hip_atomic_load(keys + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (prev == kEmpty)
      prev = atomicCAS(reinterpret_cast<unsigned long long*>(keys + h), (unsigned long long)kEmpty,
                       (unsigned long long)key);
    if (prev == kEmpty) {
      fresh = true;
      return h;
    }
    if (prev == key) return h;
    h = (h + 1) & mask;
  }
}

// slot of a key, or -1 (the table is never full: size >= 2 x keys)
__device__ __forceinline__ int hash_find(const uint64_t* keys, uint32_t mask, uint64_t key) {
  uint32_t h = hash64(key) & mask;
  for (;;) {
    const uint64_t k = keys[h];
    if (k == key) return (int)h;
    if (k == kEmpty) return -1;
    h = (h + 1) & mask;
  }
}

__device__ __forceinline__ int seg_of(const int32_t* off, int m, int i) {
  int lo = 0, hi = m;  // off[lo] <= i < off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= i) lo = mid;
    else hi = mid;
  }
  return lo;
}

// seg_of(off, m, i) for a point i at or after point i0, the same for the whole
// workgroup: points are grouped by segment, so after one search with uniform
// (scalar) loads a point's own segment is mostly the same or the next
__device__ __forceinline__ int seg_from(const int32_t* off, int m, int i0, int i) {
  int lo = seg_of(off, m, i0);
  for (int k = 0; k < 4; ++k) {
    if (lo + 1 >= m || off[lo + 1] > i) return lo;
    ++lo;
  }
  return seg_of(off, m, i);
}

// The active lanes of the wavefront that hold this lane's key (neighbouring
// points mostly share a cell, so one lane can speak for many); no memory
// access, one turn per distinct key.
__device__ __forceinline__ uint64_t same_key(uint64_t key, bool active) {
  const uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
  uint64_t pending = __ballot(active), mine = 0;
  while (pending) {
    const int leader = __builtin_ctzll(pending);
    const uint32_t l = __builtin_amdgcn_readlane(lo, leader), u = __builtin_amdgcn_readlane(hi, leader);
    const bool eq = active && lo == l && hi == u;
    const uint64_t same = __ballot(eq);
    if (eq) mine = same;
    pending &= ~same;
  }
  return mine;
}

__device__ __forceinline__ uint64_t lanes_below() {
  const int lane = threadIdx.x & 63;
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// keys[0 .. T) empty, a[0 .. na) and b[0 .. nb) zero
__global__ __launch_bounds__(256) void k_geom_init(uint64_t* keys, int64_t T, int32_t* a, int64_t na, int32_t* b,
                                                   int64_t nb) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < T || i < na || i < nb; i += (int64_t)gridDim.x * 256) {
    if (i < T) keys[i] = kEmpty;
    if (i < na) a[i] = 0;
    if (i < nb) b[i] = 0;
  }
}

// ---------------------------------------------------------------------------
// DBSCAN noise removal
// ---------------------------------------------------------------------------
// up to 64 points of a cell: sorted positions first + 64 batch ..., of count in all
struct DbItem {
  uint64_t key;
  int32_t first, count, batch, pad;
};

struct DbWork {
  uint64_t* keys;   // [T]
  int32_t* cnt;     // [T] points per cell
  int32_t* total;   // [2] sorted positions and work items given out (zeroed with cnt, which it follows)
  int2* range;      // [T] first sorted position and number of a cell's points
  int32_t* slot;    // [n] a point's cell
  int32_t* rank;    // [n] and its place among the cell's points
  DbItem* items;    // [n + n / 64 + 1]
  uint64_t* open;   // [n + n / 64 + 1] an item's points that are not core
  float4* spts;     // [n] the points by cell: coordinates, original index
  uint8_t* core;    // [n] core flag of each sorted position
  uint32_t mask;    // T - 1
};

// Files every point under its cell.  A wavefront's lanes of one cell go
// through one of them: one table access and one count per distinct cell, all
// of a wavefront's in flight together (a round trip per distinct cell, one
// after the other, and a compare-and-swap per point took 21 us for 180k
// points, this 12 us).
__global__ __launch_bounds__(256) void k_db_insert(const float* pts, const int32_t* off, int m, int n, float eps,
                                                   DbWork d) {
  const int i = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
  const bool act = i < n;
  uint64_t key = 0;
  const float* p = pts + 3 * (int64_t)min(i, n - 1);
  const float x = p[0], y = p[1], z = p[2];  // on their way while the segment is searched
  if (act) {
    const int cx = cell_of(x, eps), cy = cell_of(y, eps), cz = cell_of(z, eps);
    key = cell_key(seg_from(off, m, blockIdx.x * 256, i), cx, cy, cz);
  }
  const uint64_t same = same_key(key, act);
  const int leader = act ? __builtin_ctzll(same) : lane;
  int h = 0, base = 0;
  if (act && leader == lane) {
    bool fresh;
    h = (int)hash_insert(d.keys, d.mask, key, fresh);
    base = atomicAdd(d.cnt + h, __builtin_popcountll(same));
  }
  h = __shfl(h, leader);
  base = __shfl(base, leader);
  if (act) {
    d.slot[i] = h;
    d.rank[i] = base + __builtin_popcountll(same & lanes_below());
  }
}

// Sorted positions for every cell's points and the cells' work items, in any
// order: a block sums its 4096 slots and takes its share of both with one
// atomic.
__global__ __launch_bounds__(1024) void k_db_alloc(DbWork d, int T) {
  __shared__ uint64_t sh[16];
  __shared__ uint64_t base_sh;
  const int s0 = blockIdx.x * 4096 + 4 * threadIdx.x;
  int v[4] = {0, 0, 0, 0};
  uint64_t mine = 0;  // points low, items high
  if (s0 < T) {       // T is a multiple of 4
    const int4 q = *reinterpret_cast<const int4*>(d.cnt + s0);
    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
#pragma unroll
    for (int k = 0; k < 4; ++k) mine += (uint64_t)(uint32_t)v[k] | ((uint64_t)((v[k] + 63) >> 6) << 32);
  }
  uint64_t total;
  uint64_t at = block_exscan_1024(mine, sh, total);
  if (threadIdx.x == 0)
    base_sh = total ? atomicAdd(reinterpret_cast<unsigned long long*>(d.total), (unsigned long long)total) : 0ull;
  __syncthreads();
  at += base_sh;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (v[k] == 0) continue;
    const int first = (int)(uint32_t)at;
    d.range[s0 + k] = make_int2(first, v[k]);
    const uint32_t it = (uint32_t)(at >> 32), nb = (uint32_t)(v[k] + 63) >> 6;
    for (uint32_t q = 0; q < nb; ++q) d.items[it + q] = DbItem{d.keys[s0 + k], first, v[k], (int32_t)q, 0};
    at += (uint64_t)(uint32_t)v[k] | ((uint64_t)nb << 32);
  }
}

__global__ __launch_bounds__(256) void k_db_fill(const float* pts, int n, DbWork d) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float* p = pts + 3 * (int64_t)i;
  d.spts[d.range[d.slot[i]].x + d.rank[i]] = make_float4(p[0], p[1], p[2], __int_as_float(i));
}

// A thread per sorted position t, for grids of mostly lone points: its cell,
// then the 26 around it, look-up after look-up, until the test is settled.
template <int PASS>
__device__ __forceinline__ void db_point(const DbWork& d, int t, float e2, int min_pts, int32_t* keep) {
#pragma clang fp contract(off)
  if (PASS == 1 && d.core[t]) return;
  const float4 p = d.spts[t];
  const int i = __float_as_int(p.w);
  const uint64_t key = d.keys[d.slot[i]];
  const int x = (int)((key >> 32) & 0xFFFF) - 32768, y = (int)((key >> 16) & 0xFFFF) - 32768,
            z = (int)(key & 0xFFFF) - 32768;
  // (as in k_db_cells: at the edge of the key range each distinct cell once)
  auto rep = [](int v, int dd) { return dd > -1 && cell16(v + dd) == cell16(v + dd - 1); };
  const int want = PASS == 0 ? min_pts : 1;
  int found = 0;
  for (int k = 0; k < 27 && found < want; ++k) {
    const int c = k == 0 ? 13 : (k <= 13 ? k - 1 : k);  // the own cell first
    const int dz = c / 9 - 1, dy = c / 3 % 3 - 1, dx = c % 3 - 1;
    if (rep(z, dz) || rep(y, dy) || rep(x, dx)) continue;
    const int h = hash_find(d.keys, d.mask, cell_key((int)(key >> 48), x + dx, y + dy, z + dz));
    if (h < 0) continue;
    const int2 r = d.range[h];
    for (int j = r.x; j < r.x + r.y && found < want; ++j) {
      const float4 q = d.spts[j];
      const float ax = p.x - q.x, ay = p.y - q.y, az = p.z - q.z;
      if ((ax * ax + ay * ay) + az * az <= e2 && (PASS == 0 || d.core[j])) ++found;
    }
  }
  const int r = found >= want ? 1 : 0;
  if (PASS == 0) d.core[t] = (uint8_t)r;
  keep[i] = r;
}

// A wavefront per work item: up to 64 points of one cell against the points
// of the 27 cells around it.  Points of cells are loaded 64 at a time, one per
// lane, and each point of the item that is not settled yet is broadcast and
// tested against the 64: first the own cell's points, then, if that leaves any
// point open, those of the other 26 as one list, cells that share a face
// first, then an edge, then a corner.  Their table look-ups are made by 26 lanes at once, the
// first load of each issued before the own cell is tested.  PASS 0: core test
// (at least min_pts neighbours, itself included), keep written at the points'
// original index, the points that are not core left in the item's open mask;
// PASS 1: border test (a core neighbour) of those.  A point's result does not
// depend on the order of its neighbours.
//
// Bound by the distance tests (a broadcast, 9 operations and a count per open
// point and 64 candidates) and the chain of loads per item.  A thread per
// point that walked its 27 cells by itself, one dependent load after the
// other and as long as the slowest of its wavefront, took 213 + 62 us for 180k
// points (eps 3 cm, 8 points), this 32 + 12 us.
//
// Where most cells of a large cloud hold a point or two, there are too many
// items, each a chain of loads for a handful of tests: then a thread per point
// (db_point), whose own chain of 27 look-ups is the longer one (some 100 us) but
// runs 64 to a wavefront.  The line is where the items' chains outlast one round
// of the points' (whole call, us, items / points; points of depth images, 4
// points: 73k in 61k cells 111 / 186, 152k in 141k 199 / 223, 203k in 171k 270 /
// 276, 456k in 190k 293 / 282 and in 320k 498 / 416, 526k in 126k 250 / 378;
// uniform clouds: 100k in 88k 147 / 168, 300k in 130k 163 / 155 and in 265k 358 /
// 268); min_pts = 1 is settled by the point itself.
//
// The grid is what fits the chip at eight workgroups per CU, so the scalar
// registers must not be what keeps the eighth out: with 85 of them 73k points in
// 61k cells took 58 + 55 us, in two rounds, so 42 + 39.
template <int PASS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(80))) void k_db_cells(DbWork d, int n, float eps, int min_pts, int32_t* keep) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63;
  const int nitems = d.total[1];
  const float e2 = eps * eps;
  if (nitems > (min_pts == 1 ? 10000 : 130000 + n / 6)) {
    for (int t = blockIdx.x * 256 + threadIdx.x; t < n; t += gridDim.x * 256) db_point<PASS>(d, t, e2, min_pts, keep);
    return;
  }
  // offset + 1 of lane c's cell along each axis, two bits per lane, in the order own cell, 6 faces, 12 edges, 8 corners
  constexpr int kOrder[27][3] = {
      {1, 1, 1}, {0, 1, 1}, {2, 1, 1}, {1, 0, 1}, {1, 2, 1}, {1, 1, 0}, {1, 1, 2}, {0, 0, 1}, {0, 2, 1},
      {2, 0, 1}, {2, 2, 1}, {0, 1, 0}, {0, 1, 2}, {2, 1, 0}, {2, 1, 2}, {1, 0, 0}, {1, 0, 2}, {1, 2, 0},
      {1, 2, 2}, {0, 0, 0}, {0, 0, 2}, {0, 2, 0}, {0, 2, 2}, {2, 0, 0}, {2, 0, 2}, {2, 2, 0}, {2, 2, 2}};
  struct Packed {
    uint64_t a[3];
    constexpr Packed() : a{0, 0, 0} {
      for (int c = 0; c < 27; ++c)
        for (int x = 0; x < 3; ++x) a[x] |= (uint64_t)kOrder[c][x] << (2 * c);
    }
  };
  constexpr Packed kCells{};
  const int sh = 2 * min(lane, 26);
  const int ox = (int)((kCells.a[0] >> sh) & 3) - 1, oy = (int)((kCells.a[1] >> sh) & 3) - 1,
            oz = (int)((kCells.a[2] >> sh) & 3) - 1;
  const int stride = gridDim.x * 4;
  int it = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (it >= nitems) return;
  DbItem next = d.items[it];
  uint64_t next_open = PASS == 1 ? d.open[it] : 0ull;
  for (; it < nitems; it += stride) {
    const DbItem item = next;
    const uint64_t key = item.key;
    const int own = item.first, cnt = item.count;
    const int p0 = own + 64 * item.batch, np = min(64, cnt - 64 * item.batch);
    const uint64_t open = PASS == 0 ? (np >= 64 ? ~0ull : (1ull << np) - 1ull) : next_open;
    const int ahead = min(it + stride, nitems - 1);
    next = d.items[ahead];
    if (PASS == 1) next_open = d.open[ahead];
    if (PASS == 1 && open == 0) continue;
    const bool mine = lane < np;
    float4 pt = make_float4(0.f, 0.f, 0.f, 0.f);
    if (mine) pt = d.spts[p0 + lane];
    // the first probe of lane's neighbouring cell
    const int x = (int)((key >> 32) & 0xFFFF) - 32768, y = (int)((key >> 16) & 0xFFFF) - 32768,
              z = (int)(key & 0xFFFF) - 32768;
    // clamped cell coordinates can repeat at the edge of the key range: visit
    // each distinct neighbouring cell once (clamping is monotonic, so repeats
    // are adjacent), and the own one never again
    auto rep = [](int v, int dd) { return dd > -1 && cell16(v + dd) == cell16(v + dd - 1); };
    auto own_axis = [](int v, int dd) { return cell16(v + dd) == cell16(v); };
    const bool look = lane > 0 && lane < 27 && !rep(x, ox) && !rep(y, oy) && !rep(z, oz) &&
                      !(own_axis(x, ox) && own_axis(y, oy) && own_axis(z, oz));
    const uint64_t want = cell_key((int)(key >> 48), x + ox, y + oy, z + oz);
    uint32_t h = hash64(want) & d.mask;
    uint64_t probe = look ? d.keys[h] : kEmpty;

    uint64_t pending = open;
    int count = 0;  // lane k: neighbours of point k so far
    // every pending point against the lanes' candidates q
    auto test = [&](float4 q, bool ok) {
      for (uint64_t todo = pending; todo; todo &= todo - 1) {
        const int k = __builtin_ctzll(todo);
        const float px = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pt.x), k));
        const float py = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pt.y), k));
        const float pz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pt.z), k));
        const float dx = px - q.x, dy = py - q.y, dz = pz - q.z;
        const int c = __builtin_popcountll(__ballot(ok && (dx * dx + dy * dy) + dz * dz <= e2));
        if (lane == k) count += c;
      }
      pending &= ~__ballot(count >= (PASS == 0 ? min_pts : 1));
    };
    for (int j = lane; j - lane < cnt && pending; j += 64) {
      float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
      bool ok = j < cnt;
      if (ok) {
        q = d.spts[own + j];
        if (PASS == 1) ok = d.core[own + j] != 0;
      }
      test(q, ok);
    }
    if (pending) {
      while (probe != want && probe != kEmpty) {  // (lanes without a cell: kEmpty)
        h = (h + 1) & d.mask;
        probe = d.keys[h];
      }
      int2 c = make_int2(0, 0);
      if (probe == want) c = d.range[h];
      const int cb = c.x, cn = c.y;
      int incl = cn;
      for (int o = 1; o < 32; o <<= 1) {
        const int t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
      }
      const int total = __builtin_amdgcn_readlane(incl, 26);
      const int pre = incl - cn, adj = cb - pre;  // list entry j of the cell is sorted position adj + j
      for (int j0 = 0; j0 < total && pending; j0 += 64) {
        const int j = j0 + lane;
        int src = 0;
        for (uint64_t cells = __ballot(lane < 27 && cn > 0 && incl > j0 && pre < j0 + 64); cells; cells &= cells - 1) {
          const int c = __builtin_ctzll(cells);
          if (j >= __builtin_amdgcn_readlane(pre, c)) src = __builtin_amdgcn_readlane(adj, c);
        }
        bool ok = j < total;
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok) {
          q = d.spts[src + j];
          if (PASS == 1) ok = d.core[src + j] != 0;
        }
        test(q, ok);
      }
    }
    const int r = (int)((~pending >> lane) & 1ull);
    if (PASS == 0) {
      if (mine) {
        d.core[p0 + lane] = (uint8_t)r;
        keep[__float_as_int(pt.w)] = r;
      }
      if (lane == 0) d.open[it] = pending;
    } else if ((open >> lane) & 1ull) {
      keep[__float_as_int(pt.w)] = r;
    }
  }
}

// ---------------------------------------------------------------------------
// voxel sets
// ---------------------------------------------------------------------------
struct VoxWork {
  uint64_t* keys;   // [T] hash set of (segment, voxel)
  int32_t* vcnt;    // [m] distinct voxels per segment
  int32_t* coff;    // [m + 1] sort chunks before a segment's
  uint64_t* tmp;    // [T] each segment's keys, from the index of its first point on
  uint32_t mask;
};

// where a segment's keys begin: a segment has at most as many voxels as
// points (clamped, so that offsets out of order stay inside the table)
__device__ __forceinline__ int vox_base(const int32_t* off, int seg, int n) { return min(max(off[seg], 0), n); }

// Distinct (segment, voxel) keys, listed by segment.  Lanes of one voxel go
// through one of them, as in k_db_insert; a workgroup's new keys of a segment
// are counted in LDS and take their places with one atomic per workgroup and
// segment (points are grouped by segment; segments beyond the workgroup's
// first kVoxSegs take one per wavefront).  Voxel coordinates must fit 16 bits
// signed (|v| <= 32767): a point outside sets its segment's status to 1 and is
// left out.  180k points with 45k voxels: 15 us (32 us with a round trip per
// distinct key, and 25 us more for a pass that gathered the keys).
constexpr int kVoxSegs = 32;

__global__ __launch_bounds__(1024) void k_vox_insert(const float* pts, const int32_t* off, const int32_t* keep, int m,
                                                     int n, float v, VoxWork d, int32_t* status) {
  __shared__ int cnt[kVoxSegs], base[kVoxSegs];
  __shared__ int seg0_sh;
  const int i = blockIdx.x * 1024 + threadIdx.x, lane = threadIdx.x & 63;
  if (threadIdx.x < kVoxSegs) cnt[threadIdx.x] = 0;
  const float* p = pts + 3 * (int64_t)min(i, n - 1);
  const float x = p[0], y = p[1], z = p[2];  // on their way while the segment is searched
  bool act = i < n && (!keep || keep[i]);
  int seg = 0;
  uint64_t key = 0;
  if (i < n) seg = seg_from(off, m, blockIdx.x * 1024, i);
  if (threadIdx.x == 0) seg0_sh = seg;  // the first point of a workgroup exists
  if (act) {
    const int vx = cell_of(x, v), vy = cell_of(y, v), vz = cell_of(z, v);
    if (vx < -32767 || vx > 32767 || vy < -32767 || vy > 32767 || vz < -32767 || vz > 32767) {
      if (status) status[seg] = 1;
      act = false;
    } else {
      key = cell_key(seg, vx, vy, vz);
    }
  }
  const uint64_t same = same_key(key, act);
  bool fresh = false;
  if (act && __builtin_ctzll(same) == lane) hash_insert(d.keys, d.mask, key, fresh);
  __syncthreads();
  const int ls = seg - seg0_sh;  // >= 0: points are grouped by segment
  const bool local = ls >= 0 && ls < kVoxSegs;
  int r = 0;
  // one count per segment of the wavefront's new keys (mostly one)
  for (uint64_t pending = __ballot(fresh); pending;) {
    const int leader = __builtin_ctzll(pending);
    const int sg = __builtin_amdgcn_readlane(seg, leader);
    const uint64_t mates = __ballot(fresh && seg == sg);
    int at = 0;
    if (lane == leader) {
      if (local) at = atomicAdd(&cnt[ls], __builtin_popcountll(mates));
      else at = atomicAdd(d.vcnt + seg, __builtin_popcountll(mates));
    }
    at = __shfl(at, leader);
    if (fresh && seg == sg) r = at + __builtin_popcountll(mates & lanes_below());
    pending &= ~mates;
  }
  __syncthreads();
  if (threadIdx.x < kVoxSegs) {
    const int c = cnt[threadIdx.x];
    base[threadIdx.x] = c ? atomicAdd(d.vcnt + seg0_sh + threadIdx.x, c) : 0;
  }
  __syncthreads();
  if (fresh) d.tmp[vox_base(off, seg, n) + r + (local ? base[ls] : 0)] = key;
}

// Sorting: a workgroup per chunk of kVoxChunk keys of a segment (the chunks of
// all segments numbered through by coff).  k_vox_sort sorts a chunk, one key
// per thread, by a bitonic network whose steps inside a wavefront are lane
// exchanges; a segment of one chunk is written out at once, a longer one's
// chunks go back in place, and k_vox_merge gives each of their keys its rank:
// its place in its own chunk plus, for every other chunk, the number of that
// chunk's keys below it (a binary search with up to kVoxStage chunks in LDS).
// Keys are distinct, so every key has one rank.  One workgroup per segment
// (8192 keys in LDS, 91 steps with a barrier each) took 136 us for 36
// segments of up to 9000 voxels, these two 11 + 11 us.
constexpr int kVoxChunk = 1024;
constexpr int kVoxStage = 8;

__device__ __forceinline__ void vox_write(int32_t* o, uint64_t key) {
  o[0] = (int32_t)((key >> 32) & 0xFFFF) - 32768;
  o[1] = (int32_t)((key >> 16) & 0xFFFF) - 32768;
  o[2] = (int32_t)(key & 0xFFFF) - 32768;
}

// chunk blockIdx.x: its segment, or -1 past the last chunk
__device__ __forceinline__ int vox_chunk_seg(const int32_t* coff, int m) {
  const int b = blockIdx.x;
  return b < coff[m] ? seg_of(coff, m, b) : -1;
}

__global__ __launch_bounds__(kVoxChunk) void k_vox_sort(VoxWork d, const int32_t* off, int m, int n,
                                                        const int32_t* voff, int32_t* vox) {
  __shared__ uint64_t sk[kVoxChunk];
  const int seg = vox_chunk_seg(d.coff, m);
  if (seg < 0) return;
  const int t = threadIdx.x, c = blockIdx.x - d.coff[seg], total = voff[seg + 1] - voff[seg];
  const int len = min(kVoxChunk, total - c * kVoxChunk);
  uint64_t* chunk = d.tmp + vox_base(off, seg, n) + c * kVoxChunk;
  uint64_t key = t < len ? chunk[t] : kEmpty;
  int N = 64;
  while (N < len) N <<= 1;  // uniform; threads past N hold kEmpty and take part in their own wavefront only
  for (int size = 2; size <= N; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      uint64_t other;
      if (stride >= 64) {
        __syncthreads();
        sk[t] = key;
        __syncthreads();
        other = sk[t ^ stride];
      } else {
        other = __shfl_xor(key, stride);
      }
      const bool up = (t & size) == 0, low = (t & stride) == 0;
      if ((key > other) == (up == low)) key = other;
    }
  if (t >= len) return;
  if (total <= kVoxChunk) vox_write(vox + 3 * (int64_t)(voff[seg] + t), key);
  else chunk[t] = key;
}

__global__ __launch_bounds__(kVoxChunk) void k_vox_merge(VoxWork d, const int32_t* off, int m, int n,
                                                         const int32_t* voff, int32_t* vox) {
  __shared__ uint64_t sk[kVoxStage][kVoxChunk];
  const int seg = vox_chunk_seg(d.coff, m);
  if (seg < 0) return;
  const int t = threadIdx.x, c = blockIdx.x - d.coff[seg], total = voff[seg + 1] - voff[seg];
  if (total <= kVoxChunk) return;
  const uint64_t* keys = d.tmp + vox_base(off, seg, n);
  const int nch = (total + kVoxChunk - 1) / kVoxChunk, at = c * kVoxChunk + t;
  const bool act = at < total;
  const uint64_t key = act ? keys[at] : 0ull;
  int rank = t;
  for (int g0 = 0; g0 < nch; g0 += kVoxStage) {
    uint64_t v[kVoxStage];
#pragma unroll
    for (int g = 0; g < kVoxStage; ++g) {
      const int k = (g0 + g) * kVoxChunk + t;
      v[g] = k < total ? keys[k] : kEmpty;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kVoxStage; ++g) sk[g][t] = v[g];
    __syncthreads();
    // keys below `key` in each staged chunk (kEmpty past the end is never below); all searches advance together
    int lo[kVoxStage];
#pragma unroll
    for (int g = 0; g < kVoxStage; ++g) lo[g] = 0;
    for (int step = kVoxChunk / 2; step > 0; step >>= 1) {
#pragma unroll
      for (int g = 0; g < kVoxStage; ++g) lo[g] += sk[g][lo[g] + step - 1] < key ? step : 0;
    }
#pragma unroll
    for (int g = 0; g < kVoxStage; ++g)
      if (g0 + g != c) rank += lo[g] + (sk[g][lo[g]] < key ? 1 : 0);
  }
  if (act) vox_write(vox + 3 * (int64_t)(voff[seg] + rank), key);
}

// ---------------------------------------------------------------------------
// voxel overlap of (segment, instance) pairs
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t vox_code3(int x, int y, int z) {
  return ((uint64_t)(uint32_t)(x + (1 << 20)) << 42) | ((uint64_t)(uint32_t)(y + (1 << 20)) << 21) |
         (uint64_t)(uint32_t)(z + (1 << 20));
}

// One workgroup per (segment, instance) pair.  The longer list is staged in
// LDS, kOvPer codes per thread at a time, and every key of the shorter list is binary-
// searched there, a thread's keys together.  With boxes, every list has been
// cut into kOvParts runs of consecutive entries, and only the runs whose box
// meets the box of a run of the other list are staged or searched: the lists
// are sorted, so a run is a thin slab along x, and two lists (segments lying
// apart, or touching along one side) share few or no slabs that meet, also
// where stray voxels stretch the boxes of whole lists over the scene.  Voxel
// coordinates within +-2^20 (the voxel sets above are within +-32767).
//
// 1296 pairs of 36 x 36 lists of up to 9000 voxels: 75 us with every pair's
// longer list read by 256 threads, 25 us by boxes and 6 us to make them.  Of
// short lists a thread takes one, two or four entries: with eight always, 1600
// pairs of 200 voxels took 16.4 us a call and 10000 of 100 36, so 13.4 and 29.
// (The boxes' launch is not worth its 3 us there: 10.5 and 17 without boxes, by
// 256 threads; the host does not know the lists' lengths.)
// A wavefront goes from chunk to chunk with its keys, which are sorted as the
// chunks are; with every key loaded for every chunk 2 pairs of 100000 voxels took
// 430 us and 2 of 300000 3072, so 116 and 285, 1024 of 9000 41, so 36.
// From kOvMany pairs on a workgroup has 256 threads and half the LDS: six of
// them fit a CU, not three (registers), and the chain of dependent loads that a
// pair of short lists is (pair, offsets, boxes, entries) waits beside more others:
// 10000 pairs of 100 voxels 28 -> 18 us, of 800 32 -> 22, of 3000 41 -> 35, of
// 20000 387 -> 289.  With fewer pairs the larger workgroups are ahead on long
// lists (4096 of 9000 69 / 84 us).
constexpr int kOvParts = 32;
struct VoxBox {
  int32_t lo[3], hi[3];
};

// entries of run r of a list of n: [r n / kOvParts, (r + 1) n / kOvParts)
__device__ __forceinline__ int ov_part(int n, int r) { return (int)((int64_t)n * r / kOvParts); }

// boxes of the runs of every list, the lists of a first, then those of b; an
// empty run's box meets no other.  A workgroup per list, 32 lanes per run.
__global__ __launch_bounds__(1024) void k_vox_boxes(const int32_t* va, const int32_t* oa, int na, const int32_t* vb,
                                                    const int32_t* ob, VoxBox* boxes) {
  const int i = blockIdx.x, r = threadIdx.x >> 5;
  const int32_t* o = i < na ? oa + i : ob + (i - na);
  const int first = o[0], n = max(o[1] - first, 0), k1 = ov_part(n, r + 1);
  const int32_t* v = (i < na ? va : vb) + 3 * (int64_t)first;
  int lo[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, hi[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
#pragma unroll 4
  for (int k = ov_part(n, r) + (int)(threadIdx.x & 31); k < k1; k += 32)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int x = v[3 * (int64_t)k + d];
      lo[d] = min(lo[d], x);
      hi[d] = max(hi[d], x);
    }
#pragma unroll
  for (int d = 0; d < 3; ++d)
    for (int s = 16; s > 0; s >>= 1) {
      lo[d] = min(lo[d], __shfl_xor(lo[d], s));
      hi[d] = max(hi[d], __shfl_xor(hi[d], s));
    }
  if ((threadIdx.x & 31) == 0)
    boxes[(int64_t)i * kOvParts + r] = VoxBox{{lo[0], lo[1], lo[2]}, {hi[0], hi[1], hi[2]}};
}

constexpr int kOvPer = 8;  // entries per thread and round, loaded together (1, 2 or 4 where they cover the list)
constexpr int kOvMany = 6144;

// The runs of a list that take part, as one list of n entries: pre[r] entries
// come before run r.
struct OvRuns {
  int pre[kOvParts + 1];
  int first[kOvParts];  // place of entry 0 of the joined list if it were part of run r
};

__device__ __forceinline__ int ov_entry(const OvRuns& o, int t) {
  int r = 0;  // the last run with pre[r] <= t (runs that take no part are empty)
#pragma unroll
  for (int s = kOvParts / 2; s > 0; s >>= 1) r += o.pre[r + s] <= t ? s : 0;
  return o.first[r] + t;
}

template <int BOXES, int NT>
__global__ __launch_bounds__(NT) void k_overlap(const int32_t* va, const int32_t* oa, const int32_t* vb,
                                                 const int32_t* ob, const int32_t* pairs, int na, int nb,
                                                 const VoxBox* boxes, int32_t* out) {
  constexpr int kChunk = NT * kOvPer;
  __shared__ uint64_t sb[kChunk];
  __shared__ OvRuns runs[2];
  __shared__ uint32_t part[2];
  __shared__ int red[NT / 64];
  const int pr = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int i = pairs[2 * pr], j = pairs[2 * pr + 1];
  if (i < 0 || i >= na || j < 0 || j >= nb) {  // uniform over the workgroup
    if (tid == 0) out[pr] = 0;
    return;
  }
  const int a0 = oa[i], b0 = ob[j], la = max(oa[i + 1] - a0, 0), lb = max(ob[j + 1] - b0, 0);
  int n0 = la, n1 = lb;  // entries that take part
  if (BOXES) {
    VoxBox* box = reinterpret_cast<VoxBox*>(sb);  // [2][kOvParts], before sb holds codes
    constexpr int W = sizeof(VoxBox) / 4 * kOvParts;
    static_assert(W <= NT && kOvParts * kOvParts % NT == 0, "a load per thread and list, full rounds of tests");
    if (tid < W) {
      reinterpret_cast<int32_t*>(box)[tid] = reinterpret_cast<const int32_t*>(boxes + (int64_t)i * kOvParts)[tid];
      reinterpret_cast<int32_t*>(box)[W + tid] = reinterpret_cast<const int32_t*>(boxes + (int64_t)(na + j) * kOvParts)[tid];
    }
    if (tid < 2) part[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kOvParts * kOvParts / NT; ++u) {
      const int t = tid + NT * u;
      const VoxBox &x = box[t / kOvParts], &y = box[kOvParts + t % kOvParts];
      bool meet = true;
#pragma unroll
      for (int d = 0; d < 3; ++d) meet &= max(x.lo[d], y.lo[d]) <= min(x.hi[d], y.hi[d]);
      const uint64_t b = __ballot(meet);  // two runs of the first list by every run of the second
      if (b && lane == 0) {
        const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
        atomicOr(&part[0], ((lo ? 1u : 0u) | (hi ? 2u : 0u)) << (t / kOvParts));
        atomicOr(&part[1], lo | hi);
      }
    }
    __syncthreads();
    if (part[0] == 0) {
      if (tid == 0) out[pr] = 0;
      return;
    }
    if (wv < 2) {
      const int r = lane & (kOvParts - 1), len = wv ? lb : la;
      const int e0 = ov_part(len, r), n = (part[wv] >> r) & 1u ? ov_part(len, r + 1) - e0 : 0;
      int x = n;
      for (int o = 1; o < kOvParts; o <<= 1) {
        const int t = __shfl_up(x, o);
        if (r >= o) x += t;
      }
      if (lane < kOvParts) {
        runs[wv].pre[r] = x - n;
        runs[wv].first[r] = (wv ? b0 : a0) + e0 - (x - n);
        if (r == kOvParts - 1) runs[wv].pre[kOvParts] = x;
      }
    }
    __syncthreads();
    n0 = runs[0].pre[kOvParts];
    n1 = runs[1].pre[kOvParts];
  }
  const bool swap = n0 > n1;  // the keys are those of the list with fewer entries
  const int32_t *kl = swap ? vb : va, *tl = swap ? va : vb;
  const int kb = swap ? b0 : a0, tb = swap ? a0 : b0, nk = swap ? n1 : n0, nt = swap ? n0 : n1;
  // f with the number of entries per thread (1, 2, 4 or 8) that covers n entries, or a whole chunk
  auto per_thread = [&](int n, auto f) {
    if (n <= NT) f(std::integral_constant<int, 1>{});
    else if (n <= 2 * NT) f(std::integral_constant<int, 2>{});
    else if (n <= 4 * NT) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, kOvPer>{});
  };
  // codes of entries t0 + 64 u of a list that takes part, `past` for those beyond its n entries
  auto load = [&](auto u, const int32_t* l, int base, const OvRuns& o, int n, int t0, uint64_t past, uint64_t* code) {
#pragma unroll
    for (int k = 0; k < decltype(u)::value; ++k) {
      const int t = min(t0 + 64 * k, n - 1);
      const int32_t* v = l + 3 * (int64_t)(BOXES ? ov_entry(o, t) : base + t);
      const uint64_t c = vox_code3(v[0], v[1], v[2]);
      code[k] = t0 + 64 * k < n ? c : past;
    }
  };
  int cnt = 0;
  if (nk > 0) {
    int k0 = 0;  // where the wavefront begins: its keys of the rounds before lie below the chunk
    for (int c0 = 0; c0 < nt; c0 += kChunk) {
      int len = 0;  // staged codes, a power of two
      per_thread(nt - c0, [&](auto u) {
        constexpr int U = decltype(u)::value;
        uint64_t code[U];
        const int e0 = 64 * U * wv + lane;  // a wavefront's entries are consecutive
        load(u, tl, tb, runs[swap ? 0 : 1], nt, c0 + e0, ~1ull, code);  // past the end: above every code, equal to no key
        __syncthreads();
#pragma unroll
        for (int k = 0; k < U; ++k) sb[64 * k + e0] = code[k];
        len = NT * U;
      });
      __syncthreads();
      const uint64_t first = sb[0], last = sb[min(kChunk, nt - c0) - 1];
      for (int k1 = k0; k1 < nk; k1 += kChunk) {
        bool past = false;  // its keys of the later rounds lie above the chunk
        per_thread(nk - k1, [&](auto u) {
          constexpr int U = decltype(u)::value;
          uint64_t code[U];
          load(u, kl, kb, runs[swap ? 1 : 0], nk, k1 + 64 * U * wv + lane, ~0ull, code);
          bool any = false;
#pragma unroll
          for (int k = 0; k < U; ++k) any |= code[k] >= first && code[k] <= last;
          past = __ballot(code[0] <= last) == 0;  // the keys ascend over the lanes, then over k
          if (__ballot(code[U - 1] > last) == 0) k0 = k1 + kChunk;
          if (__ballot(any) == 0) return;
          int at[U];  // entries below the key (one less if all are); the searches advance together
#pragma unroll
          for (int k = 0; k < U; ++k) at[k] = 0;
          auto advance = [&](int step) {
#pragma unroll
            for (int k = 0; k < U; ++k) at[k] += sb[at[k] + step - 1] < code[k] ? step : 0;
          };
          if (len == kChunk) {  // unrolled
            for (int step = kChunk / 2; step > 0; step >>= 1) advance(step);
          } else {
            for (int step = len / 2; step > 0; step >>= 1) advance(step);
          }
#pragma unroll
          for (int k = 0; k < U; ++k) cnt += sb[at[k]] == code[k] ? 1 : 0;
        });
        if (past) break;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
  if (lane == 0) red[wv] = cnt;
  __syncthreads();
  if (tid == 0) {
    int t = 0;
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    out[pr] = t;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static Cam to_cam(const float* cam) {
  Cam c;
  c.fx = cam[0];
  c.fy = cam[1];
  c.cx = cam[2];
  c.cy = cam[3];
  for (int k = 0; k < 9; ++k) c.R[k] = cam[4 + k];
  for (int k = 0; k < 3; ++k) c.t[k] = cam[13 + k];
  c.dmin = cam[16];
  c.dmax = cam[17];
  return c;
}

// carves a workspace into 256-byte aligned parts
struct Carve {
  char* p;
  size_t used = 0;
  template <class T>
  T* take(size_t n) {
    T* r = reinterpret_cast<T*>(p + used);
    used += (n * sizeof(T) + 255) & ~(size_t)255;
    return r;
  }
};

static size_t bp_valid_words(int h, int w) { return (size_t)h * ((w + 63) / 64); }

size_t bp_count_ws_bytes(int m, int h, int w) {
  Carve c{nullptr};
  c.take<uint64_t>(bp_valid_words(h, w));
  c.take<int32_t>((size_t)m);
  return c.used;
}

size_t bp_write_ws_bytes(int h, int w) { return 8 * bp_valid_words(h, w); }

static void launch_bp_valid(const float* depth, int h, int w, int s, const Cam& cam, uint64_t* valid, hipStream_t st) {
  hipLaunchKernelGGL(k_bp_valid, dim3((unsigned)((bp_valid_words(h, w) + 31) / 32)), dim3(256), 0, st, depth, h, w, s, cam,
                     valid);
}

void launch_bp_count(const float* depth, const uint64_t* bits, int m, int h, int w, int s, const float* cam,
                     int32_t* offsets, char* ws, hipStream_t st) {
  Carve c{ws};
  uint64_t* valid = c.take<uint64_t>(bp_valid_words(h, w));
  int32_t* counts = c.take<int32_t>((size_t)m);
  if (m > 0) {
    launch_bp_valid(depth, h, w, s, to_cam(cam), valid, st);
    hipLaunchKernelGGL(k_bp_count, dim3(m), dim3(1024), 0, st, bits, valid, (int)bp_valid_words(h, w), counts);
  }
  hipLaunchKernelGGL(k_offsets<0>, dim3(1), dim3(1024), 0, st, counts, m, offsets, 1, nullptr);
}

void launch_bp_write(const float* depth, const uint64_t* bits, int m, int h, int w, int s, const float* cam,
                     const int32_t* offsets, float* points, char* ws, hipStream_t st) {
  if (m <= 0) return;
  if (!ws) {
    hipLaunchKernelGGL(k_bp_write, dim3(m), dim3(1024), 0, st, depth, bits, m, h, w, s, to_cam(cam), offsets, points);
    return;
  }
  uint64_t* valid = reinterpret_cast<uint64_t*>(ws);
  launch_bp_valid(depth, h, w, s, to_cam(cam), valid, st);
  const int nblk = (h + kBpRows - 1) / kBpRows, masks = std::min(m, std::max((1 << 21) / nblk, 1));
  hipLaunchKernelGGL(k_bp_write_rows, dim3(masks * nblk, (m - 1) / masks + 1), dim3(1024), 0, st, depth, bits, valid, m, h, w,
                     nblk, masks, to_cam(cam), offsets, points);
}

static uint32_t table_size(int n) {
  uint32_t T = 1024;
  while (T < 2u * (uint32_t)n) T <<= 1;
  return T;
}

static void geom_init(uint64_t* keys, int64_t T, int32_t* a, int64_t na, int32_t* b, int64_t nb, hipStream_t st) {
  const int64_t n = std::max(T, std::max(na, nb));
  hipLaunchKernelGGL(k_geom_init, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, st, keys, T, a, na,
                     b, nb);
}

static size_t dbscan_carve(char* ws, int n, DbWork& d) {
  const uint32_t T = table_size(n);
  Carve c{ws};
  d.keys = c.take<uint64_t>(T);
  d.cnt = c.take<int32_t>((size_t)T + 2);
  d.total = d.cnt + T;
  d.range = c.take<int2>(T);
  d.slot = c.take<int32_t>(n);
  d.rank = c.take<int32_t>(n);
  d.items = c.take<DbItem>((size_t)n + n / 64 + 1);
  d.open = c.take<uint64_t>((size_t)n + n / 64 + 1);
  d.spts = c.take<float4>(n);
  d.core = c.take<uint8_t>(n);
  d.mask = T - 1;
  return c.used;
}

size_t dbscan_ws_bytes(int n) {
  DbWork d;
  return dbscan_carve(nullptr, n, d);
}

void launch_dbscan(const float* pts, const int32_t* off, int m, int n, float eps, int min_pts, int32_t* keep,
                   char* ws, hipStream_t st) {
  if (n <= 0) return;
  DbWork d;
  dbscan_carve(ws, n, d);
  const int T = (int)table_size(n), nb = (n + 255) / 256;
  geom_init(d.keys, T, d.cnt, (int64_t)T + 2, nullptr, 0, st);
  hipLaunchKernelGGL(k_db_insert, dim3(nb), dim3(256), 0, st, pts, off, m, n, eps, d);
  hipLaunchKernelGGL(k_db_alloc, dim3((T + 4095) / 4096), dim3(1024), 0, st, d, T);
  hipLaunchKernelGGL(k_db_fill, dim3(nb), dim3(256), 0, st, pts, n, d);
  // at most one work item per point and one per 64; eight workgroups per CU, or
  // one per 256 points, take what there is in turn
  const int ng = std::min(nb * 64 + 1, std::max(nb, 8 * 256));
  hipLaunchKernelGGL(k_db_cells<0>, dim3(ng), dim3(256), 0, st, d, n, eps, min_pts, keep);
  hipLaunchKernelGGL(k_db_cells<1>, dim3(ng), dim3(256), 0, st, d, n, eps, min_pts, keep);
}

static size_t voxel_carve(char* ws, int n, int m, VoxWork& d) {
  const uint32_t T = table_size(n);
  Carve c{ws};
  d.keys = c.take<uint64_t>(T);
  d.tmp = c.take<uint64_t>(T);
  d.vcnt = c.take<int32_t>((size_t)m + 1);
  d.coff = c.take<int32_t>((size_t)m + 1);
  d.mask = T - 1;
  return c.used;
}

size_t voxel_ws_bytes(int n, int m) {
  VoxWork d;
  return voxel_carve(nullptr, n, m, d);
}

// distinct voxels per segment -> voff [m + 1]; their keys sorted by segment
// -> vox [voff[m]][3]
void launch_voxelize(const float* pts, const int32_t* off, const int32_t* keep, int m, int n, float v, int32_t* voff,
                     int32_t* vox, int32_t* status, char* ws, hipStream_t st) {
  VoxWork d;
  voxel_carve(ws, n, m, d);
  geom_init(d.keys, (int64_t)d.mask + 1, d.vcnt, (int64_t)m + 1, status, status ? m : 0, st);
  if (n > 0 && m > 0)
    hipLaunchKernelGGL(k_vox_insert, dim3((n + 1023) / 1024), dim3(1024), 0, st, pts, off, keep, m, n, v, d, status);
  hipLaunchKernelGGL(k_offsets<1>, dim3(1), dim3(1024), 0, st, d.vcnt, m, voff, kVoxChunk, d.coff);
  if (n <= 0 || m <= 0) return;
  // a segment of k voxels (k at most its points) has at most k / 1024 + 1 chunks
  const int nch = n / kVoxChunk + m;
  hipLaunchKernelGGL(k_vox_sort, dim3(nch), dim3(kVoxChunk), 0, st, d, off, m, n, voff, vox);
  hipLaunchKernelGGL(k_vox_merge, dim3(nch), dim3(kVoxChunk), 0, st, d, off, m, n, voff, vox);
}

// Boxes cost a launch and a pass over every list: they are made where every
// list is in more than one pair on average and the pairs are more than run at
// once (121 pairs of lists of some hundred voxels: 6 us without, 8 + 4 with;
// 1296 of up to 9000 voxels: 75 without, 25 + 6 with).
size_t overlap_ws_bytes(int na, int nb, int np) {
  return np > 512 && np > (int64_t)na + nb ? sizeof(VoxBox) * kOvParts * ((size_t)na + nb) : 0;
}

void launch_overlap(const int32_t* va, const int32_t* oa, int na, const int32_t* vb, const int32_t* ob, int nb,
                    const int32_t* pairs, int np, int32_t* out, char* ws, hipStream_t st) {
  if (np <= 0) return;
  VoxBox* boxes = reinterpret_cast<VoxBox*>(ws);
  if (boxes) hipLaunchKernelGGL(k_vox_boxes, dim3(na + nb), dim3(1024), 0, st, va, oa, na, vb, ob, boxes);
  constexpr int kPairs = 1 << 22;  // a launch's dimension holds fewer than 2^32 threads
  for (int64_t p0 = 0; p0 < np; p0 += kPairs) {
    const dim3 grid((unsigned)std::min<int64_t>(kPairs, np - p0));
    const int32_t* pp = pairs + 2 * p0;
    if (boxes && np >= kOvMany)
      hipLaunchKernelGGL((k_overlap<1, 256>), grid, dim3(256), 0, st, va, oa, vb, ob, pp, na, nb, boxes, out + p0);
    else if (boxes)
      hipLaunchKernelGGL((k_overlap<1, 512>), grid, dim3(512), 0, st, va, oa, vb, ob, pp, na, nb, boxes, out + p0);
    else
      hipLaunchKernelGGL((k_overlap<0, 512>), grid, dim3(512), 0, st, va, oa, vb, ob, pp, na, nb, nullptr, out + p0);
  }
}

}  // namespace disc
