// Open-vocabulary query over the instance embeddings (arXiv 2603.03935,
// Sec. III-C: instances are retrieved by the cosine similarity of their
// embedding with a text embedding; Sec. IV evaluates exactly this):
//   sim[j][i] = cos(text_j, emb_i)  (0 when either vector is zero)
//   for each query j, the k instances of highest similarity, higher first,
//   ties to the lower instance index.
// The similarity matrix is one dense contraction (q x m, K = e) on FP32 MFMA
// (v_mfma_f32_32x32x2f32, FP32 accumulation); the ranking is a per-query
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

// inv[r] = 1 / ||row r|| (0 for a zero row); one wavefront per row
template <int BF16>
__global__ __launch_bounds__(256) void k_invnorm(const void* x, int rows, int e, float* inv) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= rows) return;
  float a = 0.f;
  for (int c = lane * 4; c < e; c += 256) {
    const float4 v = load_row4<BF16>(x, (int64_t)r * e + c);
    a += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  if (lane == 0) inv[r] = a > 0.f ? 1.0f / __builtin_sqrtf(a) : 0.f;
}

// sim tile: 64 queries x 64 instances per workgroup (4 wavefronts of 32 x 32),
// K in steps of 16 staged through LDS.
template <int BF16>
__global__ __launch_bounds__(256) void k_sim(const float* emb, int m, const void* text, int q, int e,
                                             const float* inv_emb, const float* inv_text, float* sim) {
  constexpr int BK = 16;
  const int q0 = blockIdx.y * 64, i0 = blockIdx.x * 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wq = wv >> 1, wi = wv & 1;
  __shared__ float Ts[64][BK + 1];
  __shared__ float Ys[64][BK + 1];
  floatx16 acc = {};
  // loaders: 64 rows x 16 k = 1024 floats per operand, 4 per thread
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  for (int k0 = 0; k0 < e; k0 += BK) {
    const float4 tv = q0 + lr < q ? load_row4<BF16>(text, (int64_t)(q0 + lr) * e + k0 + lk) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 yv = i0 + lr < m ? *reinterpret_cast<const float4*>(emb + (int64_t)(i0 + lr) * e + k0 + lk)
                                  : make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    Ts[lr][lk] = tv.x; Ts[lr][lk + 1] = tv.y; Ts[lr][lk + 2] = tv.z; Ts[lr][lk + 3] = tv.w;
    Ys[lr][lk] = yv.x; Ys[lr][lk + 1] = yv.y; Ys[lr][lk + 2] = yv.z; Ys[lr][lk + 3] = yv.w;
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      const float a = Ts[32 * wq + (lane & 31)][kk + (lane >> 5)];
      const float bb = Ys[32 * wi + (lane & 31)][kk + (lane >> 5)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, bb, acc, 0, 0, 0);
    }
  }
  const int i = i0 + 32 * wi + (lane & 31);
  if (i >= m) return;
  const float yi = inv_emb[i];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int j = q0 + 32 * wq + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (j < q) sim[(int64_t)j * m + i] = acc[v] * yi * inv_text[j];
  }
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

template <int VPT, int KEYS, int FINAL>
__global__ __launch_bounds__(kTopkThreads) void k_topk(const float* sim, const uint64_t* kin, int n, int k, int nch,
                                                       uint64_t* kout, float* scores, int32_t* idx) {
  const int64_t j = blockIdx.x / nch;
  const int c0 = (int)(blockIdx.x % nch) * (kTopkThreads * VPT), tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ uint64_t gk[kTopkThreads];
  __shared__ uint64_t cand[kTopkCand];
  __shared__ uint64_t Tsh;
  __shared__ int nc_sh;
  uint64_t key[VPT];
  if (KEYS) {
    const uint64_t* row = kin + j * n;
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * kTopkThreads + tid;
      key[r] = i < n ? row[i] : 0ull;
    }
  } else {
    const float* row = sim + j * n;
    float v[VPT];
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * kTopkThreads + tid;
      v[r] = i < n ? row[i] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < VPT; ++r) {
      const int i = c0 + r * kTopkThreads + tid;
      key[r] = i < n ? rank_key(v[r], i) : 0ull;
    }
  }
  uint64_t best = 0;
#pragma unroll
  for (int r = 0; r < VPT; ++r) best = max64(best, key[r]);
  const bool wide = k > 64;  // uniform
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
    const uint64_t T = wide ? topk_threshold<kTopkThreads / 64>(gk, k) : topk_threshold<4>(gk, k);
    if (lane == 0) Tsh = T;
  }
  __syncthreads();
  const uint64_t T = max64(Tsh, 1ull);  // key 0 is no element
#pragma unroll
  for (int r = 0; r < VPT; ++r)
    if (key[r] >= T) {
      const int p = atomicAdd(&nc_sh, 1);
      if (p < kTopkCand) cand[p] = key[r];
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
  if (nc <= kTopkCand) {
    for (int c = tid; c < nc; c += kTopkThreads) {
      const uint64_t q = cand[c];
      int rank = 0;
#pragma unroll 4
      for (int i = 0; i < nc; ++i) rank += cand[i] > q ? 1 : 0;
      if (rank < k) emit(rank, q);
    }
    for (int r = nc + tid; r < k; r += kTopkThreads) emit(r, 0ull);
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
      for (int w = 0; w < kTopkThreads / 64; ++w) top = max64(top, gk[w]);
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

static void launch_topk(const float* sim, int m, int q, int k, uint64_t* ka, uint64_t* kb, float* scores, int32_t* idx,
                        hipStream_t st) {
  const int nch = topk_chunks(m, kTopkRow);
  const dim3 blk(kTopkThreads);
  if (nch == 1) {
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

// ---------------------------------------------------------------------------
// Weighted similarity heat-map of text queries over one frame's patches
// (Sec. III-C, the feature-similarity figure):
//   heat[j][p] = D_p cos(text_j, y_p),  y_p = f_p^T P,
// D of Eq. (1).  The patch tokens are projected by one FP32-MFMA contraction
// (G x E, K = C); each projected row's inverse norm is folded with D_p into
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

// Y[G][E] = tokens[G][C] P[C][E]: 64 x 64 tiles (4 wavefronts of 32 x 32),
// K in steps of 16 through LDS; TOK 0 F32, 1 BF16, 2 FP8 + scale; PB: P in BF16.
template <int TOK, int PB>
__global__ __launch_bounds__(256) void k_tokproj(const void* tok, const float* scale, int G, int C, const void* P,
                                                 int E, float* Y) {
  constexpr int BK = 16;
  const int g0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wg = wv >> 1, wn = wv & 1;
  __shared__ float As[64][BK + 1];
  __shared__ float Bs[64][BK + 1];
  floatx16 acc = {};
  const int lr = tid >> 2, lk = (tid & 3) * 4;         // A: row lr, channels lk..lk+3
  const int bk = tid >> 4, bn = (tid & 15) * 4;        // B: channel bk, columns bn..bn+3
  for (int k0 = 0; k0 < C; k0 += BK) {
    const float4 av = g0 + lr < G ? load_tok4<TOK>(tok, scale, g0 + lr, k0 + lk, C) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 bv = load_row4<PB>(P, (int64_t)(k0 + bk) * E + n0 + bn);
    __syncthreads();
    As[lr][lk] = av.x; As[lr][lk + 1] = av.y; As[lr][lk + 2] = av.z; As[lr][lk + 3] = av.w;
    Bs[bn][bk] = bv.x; Bs[bn + 1][bk] = bv.y; Bs[bn + 2][bk] = bv.z; Bs[bn + 3][bk] = bv.w;
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      const float a = As[32 * wg + (lane & 31)][kk + (lane >> 5)];
      const float b = Bs[32 * wn + (lane & 31)][kk + (lane >> 5)];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc, 0, 0, 0);
    }
  }
  // acc[v]: row 32 wg + 8 (v >> 2) + 4 (lane >> 5) + (v & 3), column 32 wn + (lane & 31)
  const int n = n0 + 32 * wn + (lane & 31);
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int g = g0 + 32 * wg + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (g < G) Y[(int64_t)g * E + n] = acc[v];
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

void launch_heatmap(const void* tok, int tok_dtype, const float* scale, int G, int C, const void* P, int p_bf16, int E,
                    const void* text, int text_bf16, int q, const float* D, float* Y, float* fac, float* inv_text,
                    float* heat, hipStream_t st) {
  const dim3 pg((G + 63) / 64, E / 64);
  auto proj = [&](auto tk, auto pb) {
    constexpr int T = decltype(tk)::value, B = decltype(pb)::value;
    hipLaunchKernelGGL((k_tokproj<T, B>), pg, dim3(256), 0, st, tok, scale, G, C, P, E, Y);
  };
  using Z = std::integral_constant<int, 0>;
  using O = std::integral_constant<int, 1>;
  using T2 = std::integral_constant<int, 2>;
  if (tok_dtype == 0) { if (p_bf16) proj(Z{}, O{}); else proj(Z{}, Z{}); }
  else if (tok_dtype == 1) { if (p_bf16) proj(O{}, O{}); else proj(O{}, Z{}); }
  else { if (p_bf16) proj(T2{}, O{}); else proj(T2{}, Z{}); }
  hipLaunchKernelGGL(k_heat_factor, dim3((G + 3) / 4), dim3(256), 0, st, Y, G, E, D, fac);
  if (text_bf16)
    hipLaunchKernelGGL(k_invnorm<1>, dim3((q + 3) / 4), dim3(256), 0, st, text, q, E, inv_text);
  else
    hipLaunchKernelGGL(k_invnorm<0>, dim3((q + 3) / 4), dim3(256), 0, st, text, q, E, inv_text);
  const dim3 grid((G + 63) / 64, (q + 63) / 64);
  if (text_bf16)
    hipLaunchKernelGGL(k_sim<1>, grid, dim3(256), 0, st, Y, G, text, q, E, fac, inv_text, heat);
  else
    hipLaunchKernelGGL(k_sim<0>, grid, dim3(256), 0, st, Y, G, text, q, E, fac, inv_text, heat);
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
  if (m > 0) hipLaunchKernelGGL(k_invnorm<0>, dim3((m + 3) / 4), dim3(256), 0, st, emb, m, e, inv_emb);
  if (text_bf16)
    hipLaunchKernelGGL(k_invnorm<1>, dim3((q + 3) / 4), dim3(256), 0, st, text, q, e, inv_text);
  else
    hipLaunchKernelGGL(k_invnorm<0>, dim3((q + 3) / 4), dim3(256), 0, st, text, q, e, inv_text);
  if (m > 0) {
    const dim3 grid((m + 63) / 64, (q + 63) / 64);
    if (text_bf16)
      hipLaunchKernelGGL(k_sim<1>, grid, dim3(256), 0, st, emb, m, text, q, e, inv_emb, inv_text, sim);
    else
      hipLaunchKernelGGL(k_sim<0>, grid, dim3(256), 0, st, emb, m, text, q, e, inv_emb, inv_text, sim);
  }
  launch_topk(sim, m, q, k, ka, kb, scores, idx, st);
}

}  // namespace disc
