// Open-vocabulary query over the instance embeddings (arXiv 2603.03935,
// Sec. III-C: instances are retrieved by the cosine similarity of their
// embedding with a text embedding; Sec. IV evaluates exactly this):
//   sim[j][i] = cos(text_j, emb_i)  (0 when either vector is zero)
//   for each query j, the k instances of highest similarity, higher first,
//   ties to the lower instance index.
// The similarity matrix is one dense contraction (q x m, K = e) on FP32 MFMA
// (FP32 accumulation); the ranking is a per-query
// selection over 64-bit keys held in registers.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "disc_device.h"

namespace disc {

typedef float floatx16 __attribute__((ext_vector_type(16)));

template <int BF16>
__device__ __forceinline__ float4 load_row4(const void* base, int64_t off) {
  if (BF16) {
    const uint2 v = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(base) + off);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xFFFF0000u));
  }
  return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + off);
}

// a row's squared norm is summed by 64 lanes, lane l taking elements 4 l .. 4 l
// + 3 of every 256, in this form, then over the lanes by xor shuffles
__device__ __forceinline__ float sq4(float4 v) { return v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w; }

__device__ __forceinline__ float inv_norm(float a) { return a > 0.f ? 1.0f / __builtin_sqrtf(a) : 0.f; }

// inv[r] = 1 / ||row r|| (0 for a zero row); one wavefront per row
template <int BF16>
__device__ __forceinline__ void invnorm_row(const void* x, int64_t r, int e, float* inv) {
  const int lane = threadIdx.x & 63;
  float a = 0.f;
  for (int c = lane * 4; c < e; c += 256) {
    a += sq4(load_row4<BF16>(x, r * e + c));
  }
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (lane == 0) inv[r] = inv_norm(a);
}

// rows 0 .. m - 1 of the result: emb; rows m .. m + q - 1: text
template <int BF16>
__global__ __launch_bounds__(256) void k_invnorms(const float* emb, int m, const void* text, int q, int e,
                                                  float* inv_emb, float* inv_text) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r < m) invnorm_row<0>(emb, r, e, inv_emb);
  else if (r - m < q) invnorm_row<BF16>(text, r - m, e, inv_text);
}

// FP32 contraction of rows of A with rows of B (both with the K elements of a
// row contiguous): a workgroup of WA x WB = 4 wavefronts computes MT WA rows
// of A by MT WB rows of B, a wavefront one MT x MT tile, MT = 32
// (v_mfma_f32_32x32x2f32) or 16 (v_mfma_f32_16x16x4f32).  FP32 MFMA adds its
// products one k after the other, each addition rounded like an fma's (checked
// bit for bit against an fma chain), so every shape gives the same bits.
//
// Bound by the FP32 matrix rate for many rows of A and by reading B for few.
// K is staged through LDS, BK at a time in two buffers.  In a step, the
// operands of each group of four MFMAs are read while the group before runs;
// before the last but one group the next step's elements, fetched a whole
// step earlier, are stored to the other buffer and the fetch of the step after
// is issued; the step's one barrier stands before the last group, whose
// operands are in registers by then.  So no wavefront waits for a load, an
// LDS read or a store with its matrix core idle.  A row's elements are stored
// in the order in which the lanes take them (all elements of one lane group
// of four consecutive MFMAs together), so an operand of four MFMAs is one
// 16-byte LDS read; the row stride BK + 4 keeps those reads free of bank
// conflicts.
//
// NORM: the squared norms of the tile's rows of A and B come with the loads
// (na, nb; valid in every lane of a row's 16 after the run), summed in the
// order of invnorm_row: a lane of it is one thread and one of four steps.
// KMB: B is stored with the rows' elements k apart (element k of row n at [k][n]):
// load_b(row, k) gives element k of rows row .. row + 3.
template <int MT, int WA, int WB, int BK, bool NORM = false, bool KMB = false>
struct GemmTile {
  static constexpr int KG = MT == 32 ? 2 : 4;  // K of one MFMA
  static constexpr int TA = MT * WA, TB = MT * WB, LD = BK + 4;
  static constexpr int QA = TA * BK / 1024, QB = TB * BK / 1024;  // 16-byte loads per thread and step
  static constexpr int NG = BK / (4 * KG);                        // operand groups of a step
  static_assert(WA * WB == 4 && QA * 1024 == TA * BK && QB * 1024 == TB * BK && NG % 2 == 0, "tile");
  typedef typename std::conditional<MT == 32, floatx16, floatx4>::type Acc;
  static constexpr int NV = MT * MT / 64;
  static_assert(!NORM || (BK == 64 && !KMB), "a row's 16 threads and four steps are invnorm_row's 64 lanes");
  alignas(16) float as[2][TA][LD];
  alignas(16) float bs[2][TB][LD];
  struct Norms {
    float a[NORM ? QA : 1], b[NORM ? QB : 1];
  };

  // rows of A and B (within the workgroup's tile) of accumulator element v of this lane
  static __device__ __forceinline__ int row_a(int v) {
    const int lane = threadIdx.x & 63, wa = (threadIdx.x >> 6) / WB;
    return MT * wa + (MT == 32 ? 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3) : 4 * (lane >> 4) + v);
  }
  static __device__ __forceinline__ int row_b() { return MT * ((threadIdx.x >> 6) % WB) + (threadIdx.x & (MT - 1)); }

  // place of elements k .. k + 3 (k % 4 == 0) in their row
  static __device__ __forceinline__ int slot(int k) {
    return MT == 32 ? (k & ~7) + ((k >> 1) & 3) : (k & ~15) + ((k >> 2) & 3);
  }
  static __device__ __forceinline__ void put(float* p, floatx4 v) {
    if (MT == 32) {
      *reinterpret_cast<float2*>(p) = make_float2(v.x, v.z);
      *reinterpret_cast<float2*>(p + 4) = make_float2(v.y, v.w);
    } else {
      p[0] = v.x; p[4] = v.y; p[8] = v.z; p[12] = v.w;
    }
  }

  // place of element k
  static __device__ __forceinline__ int place(int k) {
    return MT == 32 ? (k & ~7) + ((k >> 1) & 3) + 4 * (k & 1) : (k & ~15) + ((k >> 2) & 3) + 4 * (k & 3);
  }

  // sum over k < e of A[row_a] B[row_b]; load_a(row, k) and load_b(row, k)
  // give elements k .. k + 3 of a row of the tile (k % 4 == 0, below e)
  template <class LA, class LB>
  __device__ __forceinline__ Acc run(int e, LA load_a, LB load_b, Norms* norms = nullptr) {
    const int tid = threadIdx.x, lane = tid & 63;
    // whole vectors, so that the loads write them in place; 256 threads cover
    // 1024 / BK rows a round, so a thread's k is the same in each
    floatx4 ra[QA], rb[QB];
    constexpr int RR = 1024 / BK;
    const int kt = 4 * (tid % (BK / 4)), rt = tid / (BK / 4);
    // KMB: thread's element k and rows of load i
    auto kk = [&](int i) { return (tid + 256 * i) / (TB / 4); };
    auto kn = [&](int i) { return 4 * ((tid + 256 * i) % (TB / 4)); };
    float sa[NORM ? QA : 1][4], sb[NORM ? QB : 1][4];
    if (NORM) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int i = 0; i < QA; ++i) sa[i][j] = 0.f;
#pragma unroll
        for (int i = 0; i < QB; ++i) sb[i][j] = 0.f;
      }
    }
    auto add_sq = [](float (&s)[4], floatx4 v) {  // the step's part; the four parts move on by one
      const float t = s[0] + sq4(make_float4(v.x, v.y, v.z, v.w));
      s[0] = s[1];
      s[1] = s[2];
      s[2] = s[3];
      s[3] = t;
    };
    auto fetch = [&](int k0) {  // past the end: the last elements again
      const int k = min(k0 + kt, e - 4);
#pragma unroll
      for (int i = 0; i < QA; ++i) {
        const float4 v = load_a(rt + i * RR, k);
        ra[i] = floatx4{v.x, v.y, v.z, v.w};
      }
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        const float4 v = KMB ? load_b(kn(i), min(k0 + kk(i), e - 1)) : load_b(rt + i * RR, k);
        rb[i] = floatx4{v.x, v.y, v.z, v.w};
      }
    };
    // The loaded vectors pass through an empty asm where they are stored:
    // without it the register moves that pair up a store's elements are placed
    // right after the loads, and wait for them there.
    auto here = [](floatx4& v) { asm volatile("" : "+v"(v)); };
    auto store = [&](int buf, int k0) {
#pragma unroll
      for (int i = 0; i < QA; ++i) here(ra[i]);
#pragma unroll
      for (int i = 0; i < QB; ++i) here(rb[i]);
      if (k0 + BK > e) {  // K past e: zeros, which leave every sum's bits as they are
        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < QA; ++i) ra[i] = k0 + kt < e ? ra[i] : zero;
#pragma unroll
        for (int i = 0; i < QB; ++i) rb[i] = k0 + (KMB ? kk(i) : kt) < e ? rb[i] : zero;
      }
      if (NORM) {
#pragma unroll
        for (int i = 0; i < QA; ++i) add_sq(sa[i], ra[i]);
#pragma unroll
        for (int i = 0; i < QB; ++i) add_sq(sb[i], rb[i]);
      }
      float* pa = as[buf][rt] + slot(kt);
      float* pb = bs[buf][rt] + slot(kt);
#pragma unroll
      for (int i = 0; i < QA; ++i) put(pa + i * RR * LD, ra[i]);
#pragma unroll
      for (int i = 0; i < QB; ++i) {
        if (KMB) {
          float* q = bs[buf][kn(i)] + place(kk(i));
          q[0] = rb[i].x; q[LD] = rb[i].y; q[2 * LD] = rb[i].z; q[3 * LD] = rb[i].w;
        } else {
          put(pb + i * RR * LD, rb[i]);
        }
      }
    };
    fetch(0);
    store(0, 0);
    fetch(BK);
    __syncthreads();
    const int arow = MT * ((tid >> 6) / WB) + (lane & (MT - 1)), brow = row_b(), lg = 4 * (lane / MT);
    float4 a[2], b[2];
    auto read = [&](int buf, int g, int set) {
      a[set] = *reinterpret_cast<const float4*>(&as[buf][arow][4 * KG * g + lg]);
      b[set] = *reinterpret_cast<const float4*>(&bs[buf][brow][4 * KG * g + lg]);
    };
    Acc acc = {};
    read(0, 0, 0);
    int buf = 0;
    for (int k0 = 0; k0 < e; k0 += BK, buf ^= 1) {
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) {
          read(buf, g + 1, (g + 1) & 1);
          if (g + 2 == NG) {  // (past the last step nothing reads what is stored)
            store(buf ^ 1, k0 + BK);
            fetch(k0 + 2 * BK);
          }
        } else {
          __syncthreads();
          read(buf ^ 1, 0, (g + 1) & 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float x = (&a[g & 1].x)[s], y = (&b[g & 1].x)[s];
          if constexpr (MT == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, acc, 0, 0, 0);
          else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (NORM) {  // parts j and j + 2, then j and j + 1 (lanes 32 and 16 apart there), then the row's 16 threads
      auto total = [](const float (&s)[4]) {
        float a = (s[0] + s[2]) + (s[1] + s[3]);
        for (int o = 8; o > 0; o >>= 1) a += __shfl_xor(a, o);
        return a;
      };
#pragma unroll
      for (int i = 0; i < QA; ++i) norms->a[i] = total(sa[i]);
#pragma unroll
      for (int i = 0; i < QB; ++i) norms->b[i] = total(sb[i]);
    }
    return acc;
  }
};

// sum(r) as k_d_from_r adds it (thread t of 1024 every 1024th element, xor
// shuffles, the 16 wavefronts in order), by 256 threads
__device__ float sum_1024(const float* r, int n, float* red) {
  const int tid = threadIdx.x;
  float a[4] = {0.f, 0.f, 0.f, 0.f};
  for (int p = tid; p < n; p += 1024) {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = r[min(p + 256 * j, n - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] += p + 256 * j < n ? v[j] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    for (int o = 32; o > 0; o >>= 1) a[j] += __shfl_xor(a[j], o);
    if ((tid & 63) == 0) red[4 * j + (tid >> 6)] = a[j];
  }
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < 16; ++i) t += red[i];
  return t;
}

// sim[j][i] = (text_j . emb_i) f_i inv_text[j].  SCALE 0: f (inv_emb) and
// inv_text are given; 1: both are the inverse norms, taken from the rows as
// they are loaded (one launch and one reading of emb less: the whole call for 5
// queries over 20011 x 768 33 -> 24 us); 2: likewise, and f_i = D_i / ||emb_i|| with D of Eq. (1) from the
// m residuals r.  The workgroups of one XCD take consecutive tiles, query tiles
// first, so that a tile of instances is read from HBM by one XCD.
template <int BF16, int MT, int WA, int WB, int BK, int SCALE>
__global__ __launch_bounds__(256) void k_sim(const float* emb, int m, const void* text, int q, int e,
                                             const float* inv_emb, const float* inv_text, const float* r, float eps,
                                             float* sim, int qt) {
  typedef GemmTile<MT, WA, WB, BK, SCALE != 0> Tile;
  __shared__ Tile tile;
  __shared__ float fa[SCALE ? Tile::TA : 1], fb[SCALE ? Tile::TB : 1], red[16];
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int q0 = b % qt * Tile::TA, i0 = b / qt * Tile::TB;
  float denom = 0.f;
  if (SCALE == 2) denom = sum_1024(r, m, red) / (float)m + eps;
  typename Tile::Norms nn;
  const typename Tile::Acc acc =
      tile.run(e, [&](int x, int k) { return load_row4<BF16>(text, (int64_t)min(q0 + x, q - 1) * e + k); },
               [&](int x, int k) { return load_row4<0>(emb, (int64_t)min(i0 + x, m - 1) * e + k); }, &nn);
  if (SCALE) {
    if (threadIdx.x % 16 == 0) {
      const int x = threadIdx.x / 16;
#pragma unroll
      for (int i = 0; i < Tile::QA; ++i) fa[x + 16 * i] = inv_norm(nn.a[i]);
#pragma unroll
      for (int i = 0; i < Tile::QB; ++i) {
        const float a = nn.b[i];
        if (SCALE == 1) fb[x + 16 * i] = inv_norm(a);
        else fb[x + 16 * i] = a > 0.f ? r[min(i0 + x + 16 * i, m - 1)] / denom / __builtin_sqrtf(a) : 0.f;
      }
    }
    __syncthreads();
  }
  const int i = i0 + Tile::row_b();
  const float yi = SCALE ? fb[Tile::row_b()] : inv_emb[min(i, m - 1)];
  float tj[Tile::NV];  // all loads before the first store
#pragma unroll
  for (int v = 0; v < Tile::NV; ++v) tj[v] = SCALE ? fa[Tile::row_a(v)] : inv_text[min(q0 + Tile::row_a(v), q - 1)];
#pragma unroll
  for (int v = 0; v < Tile::NV; ++v) {
    const int j = q0 + Tile::row_a(v);
    if (j < q && i < m) sim[(int64_t)j * m + i] = acc[v] * yi * tj[v];
  }
}

// Tile by size (us of the whole query call at width 768 or 1024, 16 x 64 and 32 x
// 32 with the norms on the way, 64 x 64 with their launch; the 64 x 64 kernel
// before, K step 16 and two barriers a step, took 182 us for 1024 x 8000 alone,
// now 145):
//   q x m          5 x 20011   16 x 5000   64 x 3000   512 x 3000   1024 x 3000   1024 x 8000
//                  24/26/48    17/17/26    17/16/26    54/47/50     95/82/71      226/200/163
// Few queries are bound by reading the instances: the fewer of a tile's query
// rows are padding, the better.  The larger tile reads less through LDS per
// product but has a quarter of the workgroups and four times the chain of
// dependent MFMAs: it wins from about two tiles per CU on.
static int64_t sim_tiles(int q, int m, int ta, int tb) { return (int64_t)((q + ta - 1) / ta) * ((m + tb - 1) / tb); }
static bool sim_takes_norms(int q, int m) { return q <= 16 || sim_tiles(q, m, 64, 64) < 512; }

// SCALE as k_sim's (0: inv_emb and inv_text are given; they are unless sim_takes_norms)
template <int BF16, int SCALE>
static void launch_sim(const float* emb, int m, const void* text, int q, int e, const float* inv_emb,
                       const float* inv_text, const float* r, float eps, float* sim, hipStream_t st) {
  auto go = [&](auto kernel, int ta, int tb) {
    // queries of a launch: a grid dimension holds fewer than 2^32 threads
    const int64_t per = std::max<int64_t>(1, (1 << 23) / ((m + tb - 1) / tb)) * ta;
    for (int64_t j = 0; j < q; j += per) {
      const int n = (int)std::min<int64_t>(per, q - j);
      hipLaunchKernelGGL(kernel, dim3((unsigned)sim_tiles(n, m, ta, tb)), dim3(256), 0, st, emb, m,
                         static_cast<const char*>(text) + j * e * (BF16 ? 2 : 4), n, e, inv_emb,
                         inv_text ? inv_text + j : nullptr, r, eps, sim + j * m, (n + ta - 1) / ta);
    }
  };
  if constexpr (SCALE == 0) go(k_sim<BF16, 32, 2, 2, 32, 0>, 64, 64);
  else if constexpr (SCALE == 2) go(k_sim<BF16, 16, 2, 2, 64, 2>, 32, 32);  // (k_heat_few takes up to 16 queries)
  else if (q <= 16) go(k_sim<BF16, 16, 1, 4, 64, 1>, 16, 64);
  else go(k_sim<BF16, 16, 2, 2, 64, 1>, 32, 32);
}

// Order-preserving 64-bit key: larger score first, then smaller index.
__device__ __forceinline__ uint64_t rank_key(float s, int i) {
  const uint32_t b = __float_as_uint(s);
  const uint32_t o = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((uint64_t)o << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)i);
}

__device__ __forceinline__ float rank_score(uint64_t key) {
  const uint32_t o = (uint32_t)(key >> 32);
  return __uint_as_float((o & 0x80000000u) ? o ^ 0x80000000u : ~o);
}

__device__ __forceinline__ uint64_t max64(uint64_t a, uint64_t b) { return a > b ? a : b; }

// The k largest keys of a row, larger first.  One workgroup takes up to
// 1024 * VPT elements of a row, each thread VPT of them in registers (one
// round of loads), and
//  1. reduces them to group maxima (256 groups of four threads, or every
//     thread's own for k > 64);
//  2. one wavefront finds, bit by bit, a threshold T that at least k (and
//     usually hardly more) group maxima reach: then at least k elements do, and
//     any element below T has k larger ones;
//  3. the elements that reach T (the expected count is close to k: for k = 10
//     of 256 groups 10.2) are listed in LDS and each finds its rank by
//     counting the larger ones.
// Keys are distinct, so the result does not depend on the order of the list.
// A row laid out so that one group holds most of the large elements can list
// more than kTopkCand; it is then taken in k passes over the registers, each
// the largest key below the last.  What bounds it is latency (three barriers
// and the bit search), not the 4 bytes read per element: k dependent passes
// over the row in memory took 111 us for 1024 rows of 8000 and 118 us for 5
// rows of 20011 (k = 10), this kernel 12 and 7 us.
//
// KEYS = 0: the elements are a row of sim (element i's key from its score and
// i); 1: keys of an earlier level, 0 where there is none.  FINAL: scores and
// indices are written, (-inf, -1) past the last element; else the k keys (0
// past the last) go to kout.
constexpr int kTopkThreads = 1024;
constexpr int kTopkCand = 2048;
// Rows of up to 2048 elements, k <= 64: 256 threads, a group each, so that eight
// rows share a CU instead of two (whole calls at width 64, 1024 / 256 threads:
// 4000 rows of 300, k = 1 39.5 / 20.2 us, k = 64 44.9 / 22.4, 20000 of 2000 214 /
// 116, 64 of 2000 17 / 17; k passes over the row took 135 us for 20000 of 400
// and k = 1 at width 512, 1024 threads 228).
constexpr int kTopkFew = 256;
// elements per workgroup of the widest level-0 kernel: one level covers a row
// of up to 32768 (20011 elements: 9 us; in four chunks and a second level, 15)
constexpr int kTopkRow = 32 * kTopkThreads;
constexpr int kTopkKeys = 8 * kTopkThreads;

// T with at least k of the keys g (lane's NJ keys) at or above it, 0 if fewer
// than k are non-zero; stops once at most about k / 4 more than k are
template <int NJ>
__device__ __forceinline__ uint64_t topk_threshold(const uint64_t* gk, int k) {
  uint64_t g[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) g[j] = gk[(threadIdx.x & 63) + 64 * j];
  uint64_t T = 0;
  for (int b = 63; b >= 0; --b) {
    const uint64_t trial = T | (1ull << b);
    int c = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) c += __builtin_popcountll(__ballot(g[j] >= trial));
    if (c >= k) {
      T = trial;
      if (c <= k + (k >> 2) + 2) break;
    }
  }
  return T;
}

template <int VPT, int KEYS, int FINAL, int NT = kTopkThreads>
__global__ __launch_bounds__(NT) void k_topk(const float* sim, const uint64_t* kin, int n, int k, int nch,
                                                       uint64_t* kout, float* scores, int32_t* idx) {
  const int64_t j = blockIdx.x / nch;
  constexpr int kCand = NT == kTopkThreads ? kTopkCand : 2 * NT;
  const int c0 = (int)(blockIdx.x % nch) * (NT * VPT), tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ uint64_t gk[NT];
  __shared__ uint64_t cand[kCand];
  __shared__ uint64_t Tsh;
  __shared__ int nc_sh;
  uint64_t key[VPT];
  if (KEYS) {
    const uint64_t* row = kin + j * n;
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * NT + tid;
      key[r] = i < n ? row[i] : 0ull;
    }
  } else {
    const float* row = sim + j * n;
    float v[VPT];
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * NT + tid;
      v[r] = i < n ? row[i] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * NT + tid;
      key[r] = i < n ? rank_key(v[r], i) : 0ull;
    }
  }
  uint64_t best = 0;
#pragma unroll
  for (int r = 0; r < VPT; ++r) best = max64(best, key[r]);
  const bool wide = NT == kTopkFew || k > 64;  // uniform
  if (!wide) {
    best = max64(best, __shfl_xor(best, 1));
    best = max64(best, __shfl_xor(best, 2));
    if ((tid & 3) == 0) gk[tid >> 2] = best;
  } else {
    gk[tid] = best;
  }
  if (tid == 0) nc_sh = 0;
  __syncthreads();
  if (wv == 0) {
    const uint64_t T = wide ? topk_threshold<NT / 64>(gk, k) : topk_threshold<4>(gk, k);
    if (lane == 0) Tsh = T;
  }
  __syncthreads();
  const uint64_t T = max64(Tsh, 1ull);  // key 0 is no element
#pragma unroll
  for (int r = 0; r < VPT; ++r)
    if (key[r] >= T) {
      const int p = atomicAdd(&nc_sh, 1);
      if (p < kCand) cand[p] = key[r];
    }
  __syncthreads();
  const int nc = nc_sh;
  const int64_t o = FINAL ? j * k : (int64_t)blockIdx.x * k;
  auto emit = [&](int rank, uint64_t q) {
    if (FINAL) {
      scores[o + rank] = q ? rank_score(q) : -__builtin_inff();
      idx[o + rank] = q ? (int)(0xFFFFFFFFu - (uint32_t)q) : -1;
    } else {
      kout[o + rank] = q;
    }
  };
  if (nc <= kCand) {
    for (int c = tid; c < nc; c += NT) {
      const uint64_t q = cand[c];
      int rank = 0;
#pragma unroll 4
      for (int i = 0; i < nc; ++i) rank += cand[i] > q ? 1 : 0;
      if (rank < k) emit(rank, q);
    }
    for (int r = nc + tid; r < k; r += NT) emit(r, 0ull);
  } else {
    uint64_t last = ~0ull;
    for (int r = 0; r < k; ++r) {
      uint64_t top = 0;
#pragma unroll
      for (int i = 0; i < VPT; ++i)
        if (key[i] < last && key[i] > top) top = key[i];
      for (int s = 32; s > 0; s >>= 1) top = max64(top, __shfl_xor(top, s));
      if (lane == 0) gk[wv] = top;
      __syncthreads();
      for (int w = 0; w < NT / 64; ++w) top = max64(top, gk[w]);
      __syncthreads();
      if (tid == 0) emit(r, top);
      last = top;
    }
  }
}

static int topk_chunks(int64_t n, int per) { return (int)std::max<int64_t>(1, (n + per - 1) / per); }

// Scratch keys of the levels below the last (none for a row of one chunk):
// two buffers, each a level's output.
static void topk_scratch(int m, int q, int k, int64_t* a, int64_t* b) {
  *a = *b = 0;
  const int nch = topk_chunks(m, kTopkRow);
  if (nch == 1) return;
  *a = (int64_t)q * nch * k;
  const int nch2 = topk_chunks((int64_t)nch * k, kTopkKeys);
  if (nch2 > 1) *b = (int64_t)q * nch2 * k;
}

static void launch_topk_rows(const float* sim, int m, int q, int k, uint64_t* ka, uint64_t* kb, float* scores,
                             int32_t* idx, hipStream_t st) {
  const int nch = topk_chunks(m, kTopkRow);
  const dim3 blk(kTopkThreads);
  if (nch == 1) {
    if (m <= 8 * kTopkFew && k <= 64) {
      hipLaunchKernelGGL((k_topk<8, 0, 1, kTopkFew>), dim3(q), dim3(kTopkFew), 0, st, sim, nullptr, m, k, 1, nullptr, scores, idx);
      return;
    }
    // a row of at most 8192 leaves three quarters of the wide kernel's registers empty
    if (m <= 8 * kTopkThreads) hipLaunchKernelGGL((k_topk<8, 0, 1>), dim3(q), blk, 0, st, sim, nullptr, m, k, 1, nullptr, scores, idx);
    else hipLaunchKernelGGL((k_topk<32, 0, 1>), dim3(q), blk, 0, st, sim, nullptr, m, k, 1, nullptr, scores, idx);
    return;
  }
  hipLaunchKernelGGL((k_topk<32, 0, 0>), dim3((unsigned)(q * nch)), blk, 0, st, sim, nullptr, m, k, nch, ka, nullptr, nullptr);
  int n = nch * k;  // keys per row of the level before
  for (;;) {
    const int c = topk_chunks(n, kTopkKeys);
    if (c == 1) break;
    hipLaunchKernelGGL((k_topk<8, 1, 0>), dim3((unsigned)(q * c)), blk, 0, st, nullptr, ka, n, k, c, kb, nullptr, nullptr);
    std::swap(ka, kb);
    n = c * k;
  }
  hipLaunchKernelGGL((k_topk<8, 1, 1>), dim3(q), blk, 0, st, nullptr, ka, n, k, 1, nullptr, scores, idx);
}

// (rows one after the other in slices: a grid dimension holds fewer than 2^32
// threads; slices use the same scratch in turn)
static void launch_topk(const float* sim, int m, int q, int k, uint64_t* ka, uint64_t* kb, float* scores, int32_t* idx,
                        hipStream_t st) {
  const int per = (1 << 21) / topk_chunks(m, kTopkRow);
  for (int64_t j = 0; j < q; j += per)
    launch_topk_rows(sim + j * m, m, (int)std::min<int64_t>(per, q - j), k, ka, kb, scores + j * k, idx + j * k, st);
}

// ---------------------------------------------------------------------------
// Weighted similarity heat-map of text queries over one frame's patches
// (Sec. III-C, the feature-similarity figure):
//   heat[j][p] = D_p cos(text_j, y_p),  y_p = f_p^T P,
// D of Eq. (1).  The patch tokens are projected by one contraction (G x E, K
// = C) with FP32 sums; each projected row's inverse norm is folded with D_p into
// one per-patch factor, and the cosine contraction above (k_sim) applies it.
// ---------------------------------------------------------------------------
template <int TOK>
__device__ __forceinline__ float4 load_tok4(const void* base, const float* scale, int64_t row, int c, int C) {
  const int64_t off = row * C + c;
  if (TOK == 0) return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base) + off);
  if (TOK == 1) return load_row4<1>(base, off);
  // e4m3fn codes times the token's scale (every code value is exact in FP32)
  const uint32_t q = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(base) + off);
  const float sc = scale[row];
  const float4 x = e4m3x4_to_f32(q);
  return make_float4(x.x * sc, x.y * sc, x.z * sc, x.w * sc);
}

// Y[G][E] = tokens[G][C] P[C][E] in FP32 MFMA; TOK 0 F32, 1 BF16, 2 FP8 +
// scale; PB: P in BF16.  The first nchunk workgroups add up the tokens' channel
// sums (colsum_chunk) beside the contraction, which does not need them.  Bound
// by the FP32 matrix rate (whole call, before / now: 30 x 40 x 1024 x 768 100 / 55
// us, 78 x 138 x 1280 x 1024 with 64 queries 403 / 312; tiles of 32 x 32 took 58
// and 372).
template <int TOK, int PB>
__global__ __launch_bounds__(256) void k_tokproj(Batch b, Work wk, int nchunk, const void* tok, const float* scale,
                                                 int G, int C, const void* P, int E, float* Y) {
  if ((int)blockIdx.x < nchunk) {
    colsum_chunk<TOK>(b, wk, 0, blockIdx.x);
    return;
  }
  typedef GemmTile<32, 2, 2, 32, false, true> Tile;
  __shared__ Tile tile;
  const int t = xcd_remap(blockIdx.x - nchunk, gridDim.x - nchunk), nt = E / Tile::TB;
  const int g0 = t / nt * Tile::TA, n0 = t % nt * Tile::TB;
  const typename Tile::Acc acc =
      tile.run(C, [&](int x, int k) { return load_tok4<TOK>(tok, scale, min(g0 + x, G - 1), k, C); },
               [&](int n, int k) { return load_row4<PB>(P, (int64_t)k * E + n0 + n); });
#pragma unroll
  for (int v = 0; v < Tile::NV; ++v) {
    const int g = g0 + Tile::row_a(v);
    if (g < G) Y[(int64_t)g * E + n0 + Tile::row_b()] = acc[v];
  }
}

// The same for BF16 or FP8 tokens and a BF16 P on BF16 MFMA: the products are
// exact in FP32 either way (an e4m3 code is exact in BF16), the sums are FP32,
// and a token's scale is applied to its finished row, one rounding instead of
// one per product (error
// of the heat-map against 64 bits, rms: 1.9e-8 for either token type, 2.0e-8 and
// 2.8e-8 on FP32 MFMA).
// Tiles of 64 WM x 64, four wavefronts of 32 WM x 32, K in steps of 64 through
// two LDS buffers.  Bound by the latency of the loads when the tiles are few
// (1200 tokens: 228 workgroups, 16 steps each), so four steps are in flight
// in registers: 12 us for 1200 x 1024 x 768 with the channel sums beside it,
// 52 + 6 in FP32 tiles that loaded, stored and waited in turn.  P's rows run along n, its operand along k: a thread loads
// four k of four n and turns the block over in registers; a wavefront takes 8
// such blocks along n and 8 along k, whose 8-byte stores meet all banks.
constexpr int kProjDepth = 4;
template <int TOK, int WM>
__global__ __launch_bounds__(256) void k_tokproj16(Batch b, Work wk, int nchunk, const void* tok, const float* scale,
                                                   int G, int C, const uint16_t* P, int E, float* Y) {
  static_assert(TOK == 1 || TOK == 2, "BF16 or FP8 tokens");
  if ((int)blockIdx.x < nchunk) {
    colsum_chunk<TOK>(b, wk, 0, blockIdx.x);
    return;
  }
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  constexpr int BK = 64, LD = BK + 8, TM = 64 * WM, TN = 64;
  constexpr int QA = (TOK == 1 ? 2 : 1) * WM;  // 16-byte loads of tokens per thread and step
  __shared__ alignas(16) uint16_t as[2][TM][LD];
  __shared__ alignas(16) uint16_t bs[2][TN][LD];
  const int t = xcd_remap(blockIdx.x - nchunk, gridDim.x - nchunk), nt = E / TN;
  const int g0 = t / nt * TM, n0 = t % nt * TN;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  constexpr int PR = TOK == 1 ? 8 : 4;  // threads along a token row's step
  const int ar = tid / PR, ak = (tid % PR) * (BK / PR);
  const int bn = 4 * ((lane & 7) + 8 * (wv & 1)), bk = 4 * ((lane >> 3) + 8 * (wv >> 1));
  u32x4 ra[kProjDepth][QA];
  u32x2 rb[kProjDepth][4];
  auto fetch = [&](int s, int k0) {  // past the end: the last step again
    const int k = min(k0, C - BK);
#pragma unroll
    for (int i = 0; i < QA; ++i) {
      const int64_t at = (int64_t)min(g0 + ar + i * (256 / PR), G - 1) * C + k + ak;
      ra[s][i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(tok) + at * (TOK == 1 ? 2 : 1));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) rb[s][i] = *reinterpret_cast<const u32x2*>(P + (int64_t)(k + bk + i) * E + n0 + bn);
  };
  auto store = [&](int s, int buf) {
#pragma unroll
    for (int i = 0; i < QA; ++i) asm volatile("" : "+v"(ra[s][i]));
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(rb[s][i]));
#pragma unroll
    for (int i = 0; i < QA; ++i) {
      uint16_t* p = &as[buf][ar + i * (256 / PR)][ak];
      if (TOK == 1) {
        *reinterpret_cast<u32x4*>(p) = ra[s][i];
      } else {
        uint32_t h[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {  // 16 codes: the high halves of their FP32 values
          const float4 x = e4m3x4_to_f32(ra[s][i][j]);
          h[2 * j] = __builtin_amdgcn_perm(__float_as_uint(x.y), __float_as_uint(x.x), 0x07060302u);
          h[2 * j + 1] = __builtin_amdgcn_perm(__float_as_uint(x.w), __float_as_uint(x.z), 0x07060302u);
        }
        *reinterpret_cast<u32x4*>(p) = u32x4{h[0], h[1], h[2], h[3]};
        *reinterpret_cast<u32x4*>(p + 8) = u32x4{h[4], h[5], h[6], h[7]};
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // column bn + j: its half of the four rows' words
      const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
      const uint32_t lo = __builtin_amdgcn_perm(rb[s][1][j >> 1], rb[s][0][j >> 1], sel);
      const uint32_t hi = __builtin_amdgcn_perm(rb[s][3][j >> 1], rb[s][2][j >> 1], sel);
      *reinterpret_cast<u32x2*>(&bs[buf][bn + j][bk]) = u32x2{lo, hi};
    }
  };
  const int wm = wv >> 1, wn = wv & 1, row = lane & 31, ks = 8 * (lane >> 5);
  floatx16 acc[WM] = {};
#pragma unroll
  for (int s = 0; s < kProjDepth; ++s) fetch(s, s * BK);
  for (int kb = 0; kb < C; kb += kProjDepth * BK) {
#pragma unroll
    for (int s = 0; s < kProjDepth; ++s) {
      const int k0 = kb + s * BK, buf = s & 1;
      if (k0 >= C) break;  // uniform
      store(s, buf);
      fetch(s, k0 + kProjDepth * BK);
      __syncthreads();  // one per step: a buffer is written again two steps later
#pragma unroll
      for (int kk = 0; kk < BK; kk += 16) {
        const bf16x8 y = *reinterpret_cast<const bf16x8*>(&bs[buf][32 * wn + row][kk + ks]);
#pragma unroll
        for (int i = 0; i < WM; ++i) {
          const bf16x8 x = *reinterpret_cast<const bf16x8*>(&as[buf][32 * (WM * wm + i) + row][kk + ks]);
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc[i], 0, 0, 0);
        }
      }
    }
  }
  // acc[.][v]: row 8 (v >> 2) + 4 (lane >> 5) + (v & 3), column lane & 31
  const int n = n0 + 32 * wn + row;
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int gw = g0 + 32 * (WM * wm + i) + 4 * (lane >> 5);
    float sc[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) sc[v] = TOK == 2 ? scale[min(gw + 8 * (v >> 2) + (v & 3), G - 1)] : 1.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int g = gw + 8 * (v >> 2) + (v & 3);
      if (g < G) Y[(int64_t)g * E + n] = TOK == 2 ? acc[i][v] * sc[v] : acc[i][v];
    }
  }
}

// f[p] = D[p] / ||Y_p|| (0 for a zero row); one wavefront per row
__global__ __launch_bounds__(256) void k_heat_factor(const float* Y, int G, int E, const float* D, float* f) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= G) return;
  float a = 0.f;
  for (int c = lane * 4; c < E; c += 256) {
    const float4 v = *reinterpret_cast<const float4*>(Y + (int64_t)r * E + c);
    a += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (lane == 0) f[r] = a > 0.f ? D[r] / __builtin_sqrtf(a) : 0.f;
}

// tokens, their statistics and P to Y and r (k_mean and k_resid after the projection)
static void launch_tokproj(const Batch& b, const Work& w, const void* tok, const float* scale, int G, const void* P,
                           int p_bf16, int E, float* Y, hipStream_t st) {
  const int C = b.C, nchunk = b.nchunk, dt = b.tok_dtype;
  auto go = [&](auto kernel, int tm, int tn, auto p) {
    hipLaunchKernelGGL(kernel, dim3(nchunk + (G + tm - 1) / tm * (E / tn)), dim3(256), 0, st, b, w, nchunk, tok, scale, G,
                       C, p, E, Y);
  };
  if (dt != 0 && p_bf16) {
    const uint16_t* p = static_cast<const uint16_t*>(P);
    // taller tiles read P half as often, once there are four 64 x 64 tiles per CU
    // (whole call, 64 / 128 rows: 68 x 120 tokens x 1280 x 1024 FP8 89 / 80 us,
    // 45 x 80 x 1024 x 768 47.5 / 48.2, 30 x 40 x 1024 x 768 38.1 / 40.3)
    const bool tall = (int64_t)((G + 63) / 64) * (E / 64) >= 1024;
    if (dt == 1) { if (tall) go(k_tokproj16<1, 2>, 128, 64, p); else go(k_tokproj16<1, 1>, 64, 64, p); }
    else { if (tall) go(k_tokproj16<2, 2>, 128, 64, p); else go(k_tokproj16<2, 1>, 64, 64, p); }
    return;
  }
  auto fp32 = [&](auto tk, auto pb) { go(k_tokproj<decltype(tk)::value, decltype(pb)::value>, 64, 64, P); };
  using Z = std::integral_constant<int, 0>;
  using O = std::integral_constant<int, 1>;
  using T2 = std::integral_constant<int, 2>;
  if (dt == 1) fp32(O{}, Z{});
  else if (dt == 2) fp32(T2{}, Z{});
  else if (p_bf16) fp32(Z{}, O{});
  else fp32(Z{}, Z{});
}

// heat[j][i] = D_i cos(text_j, Y_i) for at most 16 queries: 16 patches per
// workgroup, a quarter of E per wavefront, straight into MFMA operands with all
// loads in flight, the norms on the way, the quarters added through LDS.  (The
// similarity tile, 64 patches to a workgroup, has one workgroup per 64 patches
// and walks E in 8 to 16 steps: 1200 patches x 768 15.5 us, so 8.9; error of
// the heat-map against 64 bits, rms, 1.9e-8 and 1.2e-8.)
template <int BF16>
__global__ __launch_bounds__(256) void k_heat_few(const float* Y, int G, const void* text, int q, int E, const float* r,
                                                  float eps, float* heat) {
  constexpr int NC = 16;  // pieces of 16 elements per wavefront: E <= 1024
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, row = lane & 15, g = lane >> 4;
  const int i0 = xcd_remap(blockIdx.x, gridDim.x) * 16;
  const int per = E / 4, kb = __builtin_amdgcn_readfirstlane(wv) * per;  // E is a multiple of 128: per, of 32
  const int64_t bo = (int64_t)min(i0 + row, G - 1) * E + kb + 4 * g, ao = (int64_t)min(row, q - 1) * E + kb + 4 * g;
  floatx4 a[NC], b[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int k = min(16 * j, per - 16);  // past the quarter: its last piece again
    const float4 t = load_row4<BF16>(text, ao + k);
    a[j] = floatx4{t.x, t.y, t.z, t.w};
    b[j] = *reinterpret_cast<const floatx4*>(Y + bo + k);
  }
  __shared__ float red[16];
  __shared__ alignas(16) float part[4][256];
  __shared__ float na[4][16], nb[4][16];
  const float denom = sum_1024(r, G, red) / (float)G + eps;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  float sa = 0.f, sb = 0.f;
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    floatx4 x = 16 * j < per ? a[j] : zero, y = 16 * j < per ? b[j] : zero;
    sa += sq4(make_float4(x.x, x.y, x.z, x.w));
    sb += sq4(make_float4(y.x, y.y, y.z, y.w));
    rows_to_regs(x);
    rows_to_regs(y);
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[s], y[s], acc, 0, 0, 0);
  }
  sa += __shfl_xor(sa, 32);
  sa += __shfl_xor(sa, 16);
  sb += __shfl_xor(sb, 32);
  sb += __shfl_xor(sb, 16);
  *reinterpret_cast<floatx4*>(&part[wv][4 * lane]) = acc;
  if (g == 0) {
    na[wv][row] = sa;
    nb[wv][row] = sb;
  }
  __syncthreads();
  // thread t: element v = t & 3 of lane l = t >> 2: query 4 (l >> 4) + v, patch l & 15
  const int j = 4 * (tid >> 6) + (tid & 3), n = (tid >> 2) & 15, i = i0 + n;
  if (j >= q || i >= G) return;
  const float t = (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]);
  const float ta = (na[0][j] + na[1][j]) + (na[2][j] + na[3][j]), tb = (nb[0][n] + nb[1][n]) + (nb[2][n] + nb[3][n]);
  const float f = tb > 0.f ? r[i] / denom / __builtin_sqrtf(tb) : 0.f;
  heat[(int64_t)j * G + i] = t * f * inv_norm(ta);
}

void launch_heatmap(const Batch& b, const Work& w, const void* tok, const float* scale, int G, const void* P, int p_bf16,
                    int E, const void* text, int text_bf16, int q, float eps, float* D, float* Y, float* fac, float* inv_text,
                    float* heat, hipStream_t st) {
  launch_tokproj(b, w, tok, scale, G, P, p_bf16, E, Y, st);
  launch_token_stats(b, w, G, st, true);
  if (q <= 16) {
    const dim3 grid((G + 15) / 16);
    if (text_bf16) hipLaunchKernelGGL(k_heat_few<1>, grid, dim3(256), 0, st, Y, G, text, q, E, w.r, eps, heat);
    else hipLaunchKernelGGL(k_heat_few<0>, grid, dim3(256), 0, st, Y, G, text, q, E, w.r, eps, heat);
    return;
  }
  if (sim_takes_norms(q, G)) {
    if (text_bf16) launch_sim<1, 2>(Y, G, text, q, E, nullptr, nullptr, w.r, eps, heat, st);
    else launch_sim<0, 2>(Y, G, text, q, E, nullptr, nullptr, w.r, eps, heat, st);
    return;
  }
  launch_d_from_r(w.r, G, eps, D, st);
  hipLaunchKernelGGL(k_heat_factor, dim3((G + 3) / 4), dim3(256), 0, st, Y, G, E, D, fac);
  const dim3 ng((q + 3) / 4);
  if (text_bf16) {
    hipLaunchKernelGGL(k_invnorms<1>, ng, dim3(256), 0, st, nullptr, 0, text, q, E, nullptr, inv_text);
    launch_sim<1, 0>(Y, G, text, q, E, fac, inv_text, nullptr, 0.f, heat, st);
  } else {
    hipLaunchKernelGGL(k_invnorms<0>, ng, dim3(256), 0, st, nullptr, 0, text, q, E, nullptr, inv_text);
    launch_sim<0, 0>(Y, G, text, q, E, fac, inv_text, nullptr, 0.f, heat, st);
  }
}

size_t query_ws_bytes(int m, int q, int k) {
  int64_t a, b;
  topk_scratch(m, q, k, &a, &b);
  return 8 * (size_t)(a + b) + 4 * ((size_t)m + q);
}

void launch_query(const float* emb, int m, const void* text, int text_bf16, int q, int e, int k, char* ws,
                  float* sim, float* scores, int32_t* idx, hipStream_t st) {
  int64_t na, nb;
  topk_scratch(m, q, k, &na, &nb);
  uint64_t* ka = reinterpret_cast<uint64_t*>(ws);
  uint64_t* kb = ka + na;
  float* inv_emb = reinterpret_cast<float*>(kb + nb);
  float* inv_text = inv_emb + m;
  const dim3 ng((unsigned)(((int64_t)m + q + 3) / 4));
  if (m > 0 && sim_takes_norms(q, m)) {
    if (text_bf16) launch_sim<1, 1>(emb, m, text, q, e, nullptr, nullptr, nullptr, 0.f, sim, st);
    else launch_sim<0, 1>(emb, m, text, q, e, nullptr, nullptr, nullptr, 0.f, sim, st);
  } else if (m > 0) {
    if (text_bf16) {
      hipLaunchKernelGGL(k_invnorms<1>, ng, dim3(256), 0, st, emb, m, text, q, e, inv_emb, inv_text);
      launch_sim<1, 0>(emb, m, text, q, e, inv_emb, inv_text, nullptr, 0.f, sim, st);
    } else {
      hipLaunchKernelGGL(k_invnorms<0>, ng, dim3(256), 0, st, emb, m, text, q, e, inv_emb, inv_text);
      launch_sim<0, 0>(emb, m, text, q, e, inv_emb, inv_text, nullptr, 0.f, sim, st);
    }
  }
  launch_topk(sim, m, q, k, ka, kb, scores, idx, st);
}

}  // namespace disc
