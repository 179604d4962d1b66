// Training-side forward pieces (Section 4.1: soft skip and the loss terms; Section 4.2: LoRA
// merged into the weights for inference).  Forward values only.
#pragma once
#include "prefill_attn.h"

namespace first {

// Soft skip of one layer for the prompts of a group: H = Hprev + rho * (H - Hprev), where Hprev is the stream that entered
// the layer, H holds Hprev + phi(Hprev) on entry, and rho is the router's score of Hprev (rho[j * stride] for prompt j).
// grid = rows.
__global__ void __launch_bounds__(WG) k_soft_blend(float* __restrict__ H, const float* __restrict__ Hprev,
                                                   const float* __restrict__ rho, int stride, const int* __restrict__ off, int n, int D) {
  const float r = rho[(size_t)pack_find(off, n, blockIdx.x) * stride];
  const size_t row = (size_t)blockIdx.x * D;
  for (int i = threadIdx.x * 4; i < D; i += WG * 4) {
    const float4 p = *reinterpret_cast<const float4*>(Hprev + row + i);
    float4 h = *reinterpret_cast<const float4*>(H + row + i);
    h.x = fmaf(r, h.x - p.x, p.x); h.y = fmaf(r, h.y - p.y, p.y); h.z = fmaf(r, h.z - p.z, p.z); h.w = fmaf(r, h.w - p.w, p.w);
    *reinterpret_cast<float4*>(H + row + i) = h;
  }
}

// Cross entropy of one position per workgroup: ce[j] = log(sum_v exp(l[j][v])) - l[j][target[j]],
// 0 where target[j] < 0.  Three passes over the row (max, sum of exponentials, the pick), fp32.
__global__ void __launch_bounds__(WG) k_ce_rows(const float* __restrict__ logits, const int* __restrict__ targets,
                                                float* __restrict__ ce, int V) {
  __shared__ float red[WAVES];
  const int j = blockIdx.x;
  const int t = targets[j];
  if (t < 0 || t >= V) {
    if (threadIdx.x == 0) ce[j] = 0.f;
    return;
  }
  const float* row = logits + (size_t)j * V;
  float m = -INFINITY;
  for (int v = threadIdx.x; v < V; v += WG) m = fmaxf(m, row[v]);
  m = wave_max(m);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) m = fmaxf(m, red[w]);
  float s = 0.f;
  for (int v = threadIdx.x; v < V; v += WG) s += expf(row[v] - m);
  const float tot = block_sum(s, red);
  if (threadIdx.x == 0) ce[j] = m + logf(tot) - row[t];
}

// The loss terms (Section 4.1), one workgroup per prompt of the group, fixed summation order:
//   terms[0] = L_CE  = mean of ce[j] over the positions with a target (0 when there is none)
//   terms[1] = L_Reg = sum over all router weights of w^2
//   terms[2] = L_PP  = sum_i rho[i]
//   terms[3] = L_CE + lambda * L_Reg + alpha * L_PP
__global__ void __launch_bounds__(WG) k_loss_terms(const float* __restrict__ ce, const int* __restrict__ targets, const int* __restrict__ off,
                                                   int V, const float* __restrict__ rho, int L, const float* __restrict__ router,
                                                   size_t n_router, float lambda, float alpha, float* __restrict__ terms) {
  __shared__ float red[WAVES];
  const int row0 = off[blockIdx.x] - off[0], T = off[blockIdx.x + 1] - off[blockIdx.x];
  ce += row0; targets += row0; rho += (size_t)blockIdx.x * L; terms += (size_t)blockIdx.x * 4;
  float s = 0.f, cnt = 0.f, q = 0.f, pp = 0.f;
  for (int j = threadIdx.x; j < T; j += WG) {
    const int t = targets[j];
    if (t >= 0 && t < V) { s += ce[j]; cnt += 1.f; }
  }
  // (n_router = L * D is a multiple of 8; eight 16-byte loads in flight per thread)
  for (size_t i0 = threadIdx.x * 4; i0 < n_router; i0 += WG * 32) {
    float4 w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) w[u] = *reinterpret_cast<const float4*>(router + min(i0 + (size_t)u * WG * 4, n_router - 4));
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + (size_t)u * WG * 4 < n_router) { q = fmaf(w[u].x, w[u].x, q); q = fmaf(w[u].y, w[u].y, q); q = fmaf(w[u].z, w[u].z, q); q = fmaf(w[u].w, w[u].w, q); }
  }
  for (int i = threadIdx.x; i < L; i += WG) pp += rho[i];
  const float ce_sum = block_sum(s, red);
  const float n = block_sum(cnt, red);
  const float reg = block_sum(q, red);
  const float rho_sum = block_sum(pp, red);
  if (threadIdx.x == 0) {
    const float l_ce = n > 0.f ? __fdiv_rn(ce_sum, n) : 0.f;
    terms[0] = l_ce; terms[1] = reg; terms[2] = rho_sum;
    terms[3] = l_ce + lambda * reg + alpha * rho_sum;
  }
}

// LoRA merge in place: W[row][col] += scale * sum_j Bm[row][j] * A[j][col]  (W [n, k] row-major in
// its storage type, Bm [n, r] and A [r, k] fp32).  The sum over j runs in fp32 in index order, the
// result is rounded once to the storage type.  A workgroup stages the A columns of its chunk
// (LM_COLS columns, all r rows) and the Bm rows of its row range in LDS once; a thread owns 8
// columns and walks the rows four at a time (four 16-byte loads of W in flight, every A value read
// from LDS serves four rows).  W is read and written exactly once.
constexpr int LM_COLS = 1024;      // columns per workgroup: 128 threads x 8 columns, two row groups at a time
constexpr int LM_RMAX = 32;        // largest rank (LDS: r * LM_COLS floats + the Bm rows)
constexpr int LM_RG = 4;           // rows per thread and iteration

// A matrix that the caches would not hold until it is next used goes past them (NT): what it would push out is written back meanwhile.  A program merges the
// matrices of a model once each; us through the caches / past them, bf16 of rank 8, matrices of a size in turn, 1.2 GB in all: 64 MB 31.1 / 29.6, 80 MB 37.5 / 35.6,
// 96 MB 43.3 / 41.8, 112 MB 50.4 / 48.8, 192 MB 80.7 / 78.8; rank 1 the same gains; all matrices of an 8B layer 208 / 192, of four layers 839 / 808.  The line lies at 64 MB because
// the 32 and 48 MB ones of the 8B and 3B shapes were left as they are.  What is slower past the caches is a matrix, or two, merged again at once while the 256 MB
// memory-side cache holds them: 112 MB 41 / 48, two of 64 MB in turn 24.0 / 29.3, one of 192 MB 64 / 77.  fp32 of rank 8 is 5 to 12 % slower past them at any size.
// Ranks above 8, where W waits for the sums, gain from 32 MB on, again at once or in turn: 4096 x 4096 rank 16 bf16 44.0 / 31.8, fp32 65.4 / 45.7; 14336 x 4096
// rank 32 234 / 171 and 286 / 189; only 14336 x 4096 fp32 rank 16 is slower if merged again at once (106 / 112; in turn 120 / 114).
__host__ inline bool lora_past_caches(size_t bytes, bool is_bf16, int r) { return r > 8 ? bytes >= (32u << 20) : is_bf16 && bytes >= (64u << 20); }
template <bool NT> __device__ __forceinline__ u32x4_t lora_ld(const void* p) {
  return NT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p)) : *reinterpret_cast<const u32x4_t*>(p);
}
template <bool NT> __device__ __forceinline__ void lora_st(void* p, const u32x4_t& v) {
  if (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(p));
  else *reinterpret_cast<u32x4_t*>(p) = v;
}

// One row's eight columns: W + scale * sum, rounded once.
template <typename WT, bool NT> struct LoraRow;
template <bool NT> struct LoraRow<bf16, NT> {
  u32x4_t v[1];
  __device__ __forceinline__ void load(const bf16* w) { v[0] = lora_ld<NT>(w); }
  __device__ __forceinline__ void store(bf16* w, const float (&acc)[8], float scale) const {
    u32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      o[e] = pk_bf16(fmaf(scale, acc[2 * e], __uint_as_float(v[0][e] << 16)), fmaf(scale, acc[2 * e + 1], __uint_as_float(v[0][e] & 0xffff0000u)));
    lora_st<NT>(w, o);
  }
};
template <bool NT> struct LoraRow<float, NT> {
  u32x4_t v[2];
  __device__ __forceinline__ void load(const float* w) { v[0] = lora_ld<NT>(w); v[1] = lora_ld<NT>(w + 4); }
  __device__ __forceinline__ void store(float* w, const float (&acc)[8], float scale) const {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      u32x4_t o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(fmaf(scale, acc[4 * q + e], __uint_as_float(v[q][e])));
      lora_st<NT>(w + 4 * q, o);
    }
  }
};

// Ranks up to 8 (the paper's): a thread keeps the A values of its eight columns in registers - nothing goes through LDS, no
// barrier - and walks its rows four at a time with the next four on their way; the B values of a row are the same for a
// wave and come through the scalar cache.  Ranks below 8 are padded with zeros.  Bound: HBM, W read and written once
// (14336 x 4096 / 4096 x 14336 bf16, rank 8: 59.2 / 66.9 us before, 53.5 / 51.3 now by the kernel trace = 4.4 / 4.6 TB/s; a plain
// copy runs at 4.66).
template <typename WT, bool NT>
__global__ void __launch_bounds__(WG) k_lora_merge_small(WT* __restrict__ W, const float* __restrict__ A, const float* __restrict__ Bm,
                                                         int n, int k, int r, float scale, int rows_per_wg) {
  const int col = blockIdx.x * LM_COLS + (threadIdx.x & 127) * 8, half = uni((int)(threadIdx.x >> 7));
  if (col >= k) return;                                  // k is a multiple of 8: a thread's 8 columns are in or out together
  const int half_rows = rows_per_wg / 2;                 // a multiple of LM_RG
  const int row0 = blockIdx.y * rows_per_wg + half * half_rows, row1 = min(n, row0 + half_rows);
  if (row0 >= row1) return;
  LoraRow<WT, NT> cur[LM_RG], nxt[LM_RG];
#pragma unroll
  for (int q = 0; q < LM_RG; ++q) cur[q].load(W + (size_t)min(row0 + q, row1 - 1) * k + col);
  float a[8][8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float4 a0 = make_float4(0, 0, 0, 0), a1 = a0;
    if (j < r) { a0 = *reinterpret_cast<const float4*>(A + (size_t)j * k + col); a1 = *reinterpret_cast<const float4*>(A + (size_t)j * k + col + 4); }
    a[j][0] = a0.x; a[j][1] = a0.y; a[j][2] = a0.z; a[j][3] = a0.w; a[j][4] = a1.x; a[j][5] = a1.y; a[j][6] = a1.z; a[j][7] = a1.w;
  }
  for (int rb = row0; rb < row1; rb += LM_RG) {
#pragma unroll
    for (int q = 0; q < LM_RG; ++q) nxt[q].load(W + (size_t)min(rb + LM_RG + q, row1 - 1) * k + col);   // (past the end: a row it has, not used)
#pragma unroll
    for (int q = 0; q < LM_RG; ++q) {
      const int row = min(rb + q, row1 - 1);
      const float* b = Bm + (size_t)row * r;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float bj = j < r ? b[j] : 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(bj, a[j][e], acc[e]);
      }
      if (rb + q < row1) cur[q].store(W + (size_t)row * k + col, acc, scale);
    }
#pragma unroll
    for (int q = 0; q < LM_RG; ++q) cur[q] = nxt[q];
  }
}

template <typename WT, bool NT>
__global__ void __launch_bounds__(WG) k_lora_merge(WT* __restrict__ W, const float* __restrict__ A, const float* __restrict__ Bm,
                                                   int n, int k, int r, float scale, int rows_per_wg) {
  extern __shared__ float lm_lds[];                      // A tile [r][LM_COLS], then Bm rows [rows_per_wg][r] (zero beyond n)
  float* a_lds = lm_lds;
  float* b_lds = lm_lds + r * LM_COLS;
  const int c0 = blockIdx.x * LM_COLS;
  const int row0 = blockIdx.y * rows_per_wg, row1 = min(n, row0 + rows_per_wg);
  for (int i = threadIdx.x; i < r * LM_COLS; i += WG) {
    const int j = i / LM_COLS, c = c0 + i % LM_COLS;
    a_lds[i] = c < k ? A[(size_t)j * k + c] : 0.f;
  }
  for (int i = threadIdx.x; i < rows_per_wg * r; i += WG)
    b_lds[i] = (row0 + i / r) < row1 ? Bm[(size_t)row0 * r + i] : 0.f;
  __syncthreads();
  const int tc = (threadIdx.x & 127) * 8, half = threadIdx.x >> 7;
  const int col = c0 + tc;
  if (col >= k) return;                                  // k is a multiple of 8: a thread's 8 columns are in or out together
  for (int rb = half * LM_RG; row0 + rb < row1; rb += 2 * LM_RG) {
    LoraRow<WT, NT> raw[LM_RG];
#pragma unroll
    for (int q = 0; q < LM_RG; ++q) raw[q].load(W + (size_t)min(row0 + rb + q, row1 - 1) * k + col);   // rows past the end re-read the last one and are not stored
    float acc[LM_RG][8];
#pragma unroll
    for (int q = 0; q < LM_RG; ++q)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[q][e] = 0.f;
    for (int j = 0; j < r; ++j) {
      const float4 a0 = *reinterpret_cast<const float4*>(a_lds + j * LM_COLS + tc);
      const float4 a1 = *reinterpret_cast<const float4*>(a_lds + j * LM_COLS + tc + 4);
      const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
      for (int q = 0; q < LM_RG; ++q) {
        const float bj = b_lds[(rb + q) * r + j];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[q][e] = fmaf(bj, a[e], acc[q][e]);
      }
    }
#pragma unroll
    for (int q = 0; q < LM_RG; ++q) {
      const int row = row0 + rb + q;
      if (row >= row1) break;
      raw[q].store(W + (size_t)row * k + col, acc[q], scale);
    }
  }
}

}  // namespace first
