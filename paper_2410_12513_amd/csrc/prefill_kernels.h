// Prefill kernels: every layer runs on the whole prompt (Section 4.3 item 1), the routers
// are scored on the stream entering each layer (Section 4.1), KV of all layers is written.
#pragma once
#include "common.h"

namespace first {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

// hi = bf16(x), lo = bf16(x - hi) for a pair
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = pk_bf16(a, b);
  lo = pk_bf16(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

// Prompts go through the layers in groups, packed row after row.
// The prompts of one group: rows off[j] - off[0] .. of sequence b0 + j, padded rows from poff[j] - poff[0].
struct PromptPack {
  const int *off, *poff;
  int n, b0;
  const int* pt;               // page tables [max_batch][max_pages]
  int max_pages;
};
// Index j with o[j] <= o[0] + row < o[j + 1].
__device__ __forceinline__ int pack_find(const int* o, int n, int row) {
  int lo = 0, hi = n;
  const int at = o[0] + row;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (o[mid] <= at) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ float4 keep4(float4 v, bool in) { return make_float4(in ? v.x : 0.f, in ? v.y : 0.f, in ? v.z : 0.f, in ? v.w : 0.f); }

// H[t] = E[ids[t]] widened to fp32.  grid = T.
template <typename WT>
__global__ void __launch_bounds__(WG) k_embed_rows(const int* __restrict__ ids, const WT* __restrict__ E,
                                                   float* __restrict__ H, int D, int V) {
  const int t = blockIdx.x;
  int tok = ids[t];
  tok = min(max(tok, 0), V - 1);
  const WT* row = E + (size_t)tok * D;
  for (int k = threadIdx.x; k < D; k += WG) H[(size_t)t * D + k] = to_f32(row[k]);
}

// cs[t][i] = (cos, sin)(t * theta_i), angle formed in fp64.  grid covers T*half threads.
__global__ void __launch_bounds__(WG) k_rope_table(const double* __restrict__ theta, float2* __restrict__ cs,
                                                   int T, int half) {
  const int i = blockIdx.x * WG + threadIdx.x;
  if (i >= T * half) return;
  const int t = i / half, d = i - t * half;
  const double a = (double)t * theta[d];
  cs[i] = make_float2((float)cos(a), (float)sin(a));
}

// One wave per token: x = RMSNorm(H[t]; gain) in the GEMM input type, and, if rw is given,
// sig[t] = sigmoid(rw . H[t]) on the raw stream (router, Section 4.1).  grid = ceil(T/4).
template <typename XT>
__global__ void __launch_bounds__(WG) k_rmsnorm_router(const float* __restrict__ H, const float* __restrict__ gain,
                                                       const float* __restrict__ rw, XT* __restrict__ x,
                                                       float* __restrict__ sig, int T, int D, float eps,
                                                       bf16* __restrict__ xh = nullptr, bf16* __restrict__ xl = nullptr) {
  const int t = blockIdx.x * WAVES + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= T) return;
  const float* row = H + (size_t)t * D;
  // Eight 16-byte pieces of the row per lane and round, all requested before the first is used (one piece per round
  // is one memory round trip per round); same order of additions as a piece-by-piece loop.
  constexpr int RB = 8;
  float ss = 0.f, dot = 0.f;
  for (int k0 = lane * 4; k0 < D; k0 += 256 * RB) {
    float4 v[RB], w[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int k = min(k0 + 256 * u, D - 4);
      v[u] = *reinterpret_cast<const float4*>(row + k);
      w[u] = rw ? *reinterpret_cast<const float4*>(rw + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      if (k0 + 256 * u < D) {
        ss = fmaf(v[u].x, v[u].x, ss); ss = fmaf(v[u].y, v[u].y, ss); ss = fmaf(v[u].z, v[u].z, ss); ss = fmaf(v[u].w, v[u].w, ss);
        dot = fmaf(v[u].x, w[u].x, dot); dot = fmaf(v[u].y, w[u].y, dot); dot = fmaf(v[u].z, w[u].z, dot); dot = fmaf(v[u].w, w[u].w, dot);
      }
    }
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)D + eps);
#pragma unroll 4
  for (int k = lane * 4; k < D; k += 256) {
    const float4 v = *reinterpret_cast<const float4*>(row + k);
    const float4 g = *reinterpret_cast<const float4*>(gain + k);
    const float y[4] = {v.x * g.x * r, v.y * g.y * r, v.z * g.z * r, v.w * g.w * r};
    if (xh) {                                      // split for the matrix cores: y = hi + lo
      uint16_t hi[4], lo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) { hi[e] = f2bf(y[e]); lo[e] = f2bf(y[e] - bf2f(hi[e])); }
      *reinterpret_cast<uint2*>(xh + (size_t)t * D + k) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
      *reinterpret_cast<uint2*>(xl + (size_t)t * D + k) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
    } else {
      XT* o = x + (size_t)t * D + k;
      o[0] = from_f32<XT>(y[0]); o[1] = from_f32<XT>(y[1]); o[2] = from_f32<XT>(y[2]); o[3] = from_f32<XT>(y[3]);
    }
  }
  if (rw) {
    dot = wave_sum(dot);
    if (lane == 0) sig[t] = sigmoidf(dot);
  }
}

// The same with a workgroup per token, for rows long enough to give every thread several pieces: at 1024 tokens a wave per
// token is one wave per SIMD, and reads the row twice.  The first 4096 elements of the row stay in registers between the
// sums and the scaling.  Bound: HBM / latency (1024 x 4096, 33 MB: 17.6 -> 9.0 us,
// kernel trace).
template <typename XT>
__global__ void __launch_bounds__(WG) k_rmsnorm_router_wide(const float* __restrict__ H, const float* __restrict__ gain,
                                                            const float* __restrict__ rw, XT* __restrict__ x, float* __restrict__ sig,
                                                            int D, float eps, bf16* __restrict__ xh, bf16* __restrict__ xl) {
  __shared__ float2 red[WAVES];
  constexpr int RB = 4;
  const int t = blockIdx.x, tid = threadIdx.x;
  const float* row = H + (size_t)t * D;
  float4 v[RB];
  float ss = 0.f, dot = 0.f;
  auto add = [&](const float4& a, const float4& w) __attribute__((always_inline)) {
    ss = fmaf(a.x, a.x, ss); ss = fmaf(a.y, a.y, ss); ss = fmaf(a.z, a.z, ss); ss = fmaf(a.w, a.w, ss);
    dot = fmaf(a.x, w.x, dot); dot = fmaf(a.y, w.y, dot); dot = fmaf(a.z, w.z, dot); dot = fmaf(a.w, w.w, dot);
  };
  const float4 zero = make_float4(0, 0, 0, 0);
  {
    float4 w[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int k = tid * 4 + u * WG * 4;
      v[u] = keep4(*reinterpret_cast<const float4*>(row + min(k, D - 4)), k < D);
      w[u] = zero;
      if (rw) w[u] = keep4(*reinterpret_cast<const float4*>(rw + min(k, D - 4)), k < D);
    }
#pragma unroll
    for (int u = 0; u < RB; ++u) add(v[u], w[u]);
  }
  for (int k = tid * 4 + RB * WG * 4; k < D; k += WG * 4) {
    float4 w = zero;
    if (rw) w = *reinterpret_cast<const float4*>(rw + k);
    add(*reinterpret_cast<const float4*>(row + k), w);
  }
  ss = wave_sum(ss); dot = wave_sum(dot);
  if ((tid & 63) == 0) red[tid >> 6] = make_float2(ss, dot);
  __syncthreads();
  ss = 0.f; dot = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) { ss += red[w].x; dot += red[w].y; }
  const float r = 1.0f / sqrtf(ss / (float)D + eps);
  auto put = [&](int k, const float4& a) __attribute__((always_inline)) {
    const float4 g = *reinterpret_cast<const float4*>(gain + k);
    const float y[4] = {a.x * g.x * r, a.y * g.y * r, a.z * g.z * r, a.w * g.w * r};
    if (xh) {                                      // split for the matrix cores: y = hi + lo
      uint2 hi, lo;
      split_pair(y[0], y[1], hi.x, lo.x); split_pair(y[2], y[3], hi.y, lo.y);
      *reinterpret_cast<uint2*>(xh + (size_t)t * D + k) = hi;
      *reinterpret_cast<uint2*>(xl + (size_t)t * D + k) = lo;
    } else {
      XT* o = x + (size_t)t * D + k;
      o[0] = from_f32<XT>(y[0]); o[1] = from_f32<XT>(y[1]); o[2] = from_f32<XT>(y[2]); o[3] = from_f32<XT>(y[3]);
    }
  };
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int k = tid * 4 + u * WG * 4;
    if (k < D) put(k, v[u]);
  }
  for (int k = tid * 4 + RB * WG * 4; k < D; k += WG * 4) put(k, *reinterpret_cast<const float4*>(row + k));
  if (rw && tid == 0) sig[t] = sigmoidf(dot);
}

// rho = mean_t sig[t] (fixed summation order); mask = (rho >= 0.5).  One workgroup per prompt j of the group (blockIdx.x; rows
// off[j] - off[0] .. of sig) and layer i (blockIdx.y; sig + i * sig_pitch); results at rho / mask + j * stride + i.  (A thread requests eight of its values before it adds the first: one
// after the other took 20 us at 16384 tokens.)
__global__ void __launch_bounds__(WG) k_router_reduce(const float* __restrict__ sig, size_t sig_pitch, const int* __restrict__ off,
                                                      float* __restrict__ rho, uint8_t* __restrict__ mask, int stride) {
  __shared__ float red[WAVES];
  const int j = blockIdx.x, T = off[j + 1] - off[j];
  sig += blockIdx.y * sig_pitch + (off[j] - off[0]);
  float s = 0.f;
  for (int t0 = threadIdx.x; t0 < T; t0 += 8 * WG) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = sig[min(t0 + u * WG, T - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (t0 + u * WG < T) s += v[u];
  }
  const float tot = block_sum(s, red);
  if (threadIdx.x == 0) {
    const float r = __fdiv_rn(tot, (float)T);
    rho[(size_t)j * stride + blockIdx.y] = r;
    mask[(size_t)j * stride + blockIdx.y] = (r >= 0.5f) ? 1 : 0;
  }
}

// Last position of every prompt of the group: H row -> residual slot of its sequence (and hidden_out), length -> len.
__global__ void __launch_bounds__(WG) k_last_rows(const float* __restrict__ H, const int* __restrict__ off, float* __restrict__ h,
                                                  float* __restrict__ hidden_out, int* __restrict__ len, int D) {
  const int j = blockIdx.x, T = off[j + 1] - off[j];
  const float* src = H + (size_t)(off[j + 1] - off[0] - 1) * D;
  for (int k = threadIdx.x; k < D; k += WG) {
    const float v = src[k];
    h[(size_t)j * D + k] = v;
    if (hidden_out) hidden_out[(size_t)j * D + k] = v;
  }
  if (threadIdx.x == 0) len[j] = T;
}

// kept = ascending indices of set mask bytes; one wave per sequence (ballot + popcount).
__global__ void __launch_bounds__(64) k_compact(const uint8_t* __restrict__ mask, int L, int* __restrict__ kept,
                                                int* __restrict__ n_kept) {
  const int b = blockIdx.x, lane = threadIdx.x;
  int base = 0;
  for (int i0 = 0; i0 < L; i0 += 64) {
    const int i = i0 + lane;
    const bool on = (i < L) && mask[(size_t)b * L + i] != 0;
    const unsigned long long bal = __ballot(on);
    if (on) kept[(size_t)b * L + base + __popcll(bal & ((1ull << lane) - 1ull))] = i;
    base += __popcll(bal);
  }
  for (int i = base + lane; i < L; i += 64) kept[(size_t)b * L + i] = -1;
  if (lane == 0) n_kept[b] = base;
}

// ---------------------------------------------------------------------------------------
// C[M,N] (+)= A[M,K] . W[N,K]^T, bf16 inputs, fp32 accumulate on the matrix cores.
// 128x128 tile per workgroup, 4 waves of 64x64 (2x2 MFMA 32x32x16), K step 64, operands
// staged through LDS with the next tile prefetched into registers.
constexpr int GB_M = 128, GB_N = 128, GB_K = 64, GB_PITCH = GB_K + 8;

__global__ void __launch_bounds__(WG) k_gemm_nt_bf16(const bf16* __restrict__ A, const bf16* __restrict__ W,
                                                     float* __restrict__ C, int M, int N, int K, int accumulate) {
  __shared__ __align__(16) uint16_t sA[GB_M * GB_PITCH];
  __shared__ __align__(16) uint16_t sB[GB_N * GB_PITCH];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int m0 = blockIdx.y * GB_M, n0 = blockIdx.x * GB_N;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  floatx16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  uint4 ra[4], rb[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      const int k = k0 + kc;
      ra[i] = make_uint4(0, 0, 0, 0);
      rb[i] = make_uint4(0, 0, 0, 0);
      if (k < K) {
        if (m0 + row < M) ra[i] = *reinterpret_cast<const uint4*>(A + (size_t)(m0 + row) * K + k);
        if (n0 + row < N) rb[i] = *reinterpret_cast<const uint4*>(W + (size_t)(n0 + row) * K + k);
      }
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      *reinterpret_cast<uint4*>(sA + row * GB_PITCH + kc) = ra[i];
      *reinterpret_cast<uint4*>(sB + row * GB_PITCH + kc) = rb[i];
    }
  };

  fetch(0);
  for (int k0 = 0; k0 < K; k0 += GB_K) {
    __syncthreads();
    stash();
    __syncthreads();
    if (k0 + GB_K < K) fetch(k0 + GB_K);
#pragma unroll
    for (int kk = 0; kk < GB_K; kk += 16) {
      bf16x8_t a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *reinterpret_cast<const bf16x8_t*>(sA + (wm + i * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3));
        b[i] = *reinterpret_cast<const bf16x8_t*>(sB + (wn + i * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  // D layout of the 32x32 MFMA: lane -> column (lane & 31); register r -> row
  // 8*(r/4) + 4*(lane/32) + r%4.
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < M && col < N) {
          float* c = C + (size_t)row * N + col;
          *c = accumulate ? *c + acc[i][j][r] : acc[i][j][r];
        }
      }
    }
}

// Same contraction with fp32 activations A and bf16 weights W.  Each activation is split into
// two bf16 numbers, a = hi + lo with hi = bf16(a) and lo = bf16(a - hi), and both parts go
// through the matrix cores against the same weight tile, so the product carries about 16
// mantissa bits of the activation instead of 8 (the weights are bf16 exactly).  This keeps
// the prompt's hidden states, KV and first-token logits close to full-precision arithmetic
// at twice the matrix-core work.
__global__ void __launch_bounds__(WG) k_gemm_nt_bf16_split(const float* __restrict__ A, const bf16* __restrict__ W,
                                                           float* __restrict__ C, int M, int N, int K, int accumulate) {
  __shared__ __align__(16) uint16_t sAh[GB_M * GB_PITCH];
  __shared__ __align__(16) uint16_t sAl[GB_M * GB_PITCH];
  __shared__ __align__(16) uint16_t sB[GB_N * GB_PITCH];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int m0 = blockIdx.y * GB_M, n0 = blockIdx.x * GB_N;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
  floatx16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  float4 ra[4][2];
  uint4 rb[4];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      const int k = k0 + kc;
      ra[i][0] = make_float4(0, 0, 0, 0); ra[i][1] = make_float4(0, 0, 0, 0);
      rb[i] = make_uint4(0, 0, 0, 0);
      if (k < K) {
        if (m0 + row < M) {
          ra[i][0] = *reinterpret_cast<const float4*>(A + (size_t)(m0 + row) * K + k);
          ra[i][1] = *reinterpret_cast<const float4*>(A + (size_t)(m0 + row) * K + k + 4);
        }
        if (n0 + row < N) rb[i] = *reinterpret_cast<const uint4*>(W + (size_t)(n0 + row) * K + k);
      }
    }
  };
  auto split2 = [](float a, float b, uint32_t& hi, uint32_t& lo) {
    const uint32_t ha = f2bf(a), hb = f2bf(b);
    hi = ha | (hb << 16);
    lo = (uint32_t)f2bf(a - bf2f(ha)) | ((uint32_t)f2bf(b - bf2f(hb)) << 16);
  };
  auto stash = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      uint4 h, l;
      split2(ra[i][0].x, ra[i][0].y, h.x, l.x); split2(ra[i][0].z, ra[i][0].w, h.y, l.y);
      split2(ra[i][1].x, ra[i][1].y, h.z, l.z); split2(ra[i][1].z, ra[i][1].w, h.w, l.w);
      *reinterpret_cast<uint4*>(sAh + row * GB_PITCH + kc) = h;
      *reinterpret_cast<uint4*>(sAl + row * GB_PITCH + kc) = l;
      *reinterpret_cast<uint4*>(sB + row * GB_PITCH + kc) = rb[i];
    }
  };

  fetch(0);
  for (int k0 = 0; k0 < K; k0 += GB_K) {
    __syncthreads();
    stash();
    __syncthreads();
    if (k0 + GB_K < K) fetch(k0 + GB_K);
#pragma unroll
    for (int kk = 0; kk < GB_K; kk += 16) {
      bf16x8_t ah[2], al[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int ao = (wm + i * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3);
        ah[i] = *reinterpret_cast<const bf16x8_t*>(sAh + ao);
        al[i] = *reinterpret_cast<const bf16x8_t*>(sAl + ao);
        b[i] = *reinterpret_cast<const bf16x8_t*>(sB + (wn + i * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], b[j], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = n0 + wn + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < M && col < N) {
          float* c = C + (size_t)row * N + col;
          *c = accumulate ? *c + acc[i][j][r] : acc[i][j][r];
        }
      }
    }
}

// The same split-precision contraction with the activations already split by their producer
// (Ah + Al, bf16 each): no conversion work here, which otherwise repeats once per column tile.
// A 16-byte global load whose destination the compiler must treat as in use from here on (it is written when the load
// lands), a wait that leaves the N youngest loads of the wave outstanding, and the point from which a destination
// may be read.  A kernel using these must not spill registers (see build.py).
__device__ __forceinline__ void pf_issue16(u32x4_t& v, const void* p) {
  asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(v) : "v"(p) : "memory");
}
template <int N> __device__ __forceinline__ void pf_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void pf_use(u32x4_t& v) { asm volatile("" : "+v"(v)); }

// BM x BN output tile per workgroup, the four waves arranged WGM x WGN over it (wave tile = (BM / WGM) x (BN / WGN),
// a multiple of 32 x 32 each way).
// GU: the B tile is BN / 2 rows of W (gate) followed by the same BN / 2 rows of W2 (up); instead of storing C the
// epilogue forms SiLU(gate) * up for the tile's BM x BN / 2 outputs and writes them split into zh + zl ([M, N] bf16 each).
template <int BM, int BN, int WGM, int WGN, int NSTG = 2, bool GU = false>
__device__ __forceinline__ void gemm_nt_bf16_hl_tile(const bf16* __restrict__ Ah, const bf16* __restrict__ Al,
                                                     const bf16* __restrict__ W, float* __restrict__ C, int M, int N,
                                                     int K, int accumulate, int m0, int n0,
                                                     const bf16* __restrict__ W2 = nullptr, bf16* __restrict__ zh = nullptr,
                                                     bf16* __restrict__ zl = nullptr) {
  static_assert(WGM * WGN == WAVES, "four waves");
  constexpr int TM = BM / WGM, TN = BN / WGN, IM = TM / 32, JN = TN / 32;
  constexpr int VA = BM * 8 / WG, VB = BN * 8 / WG;            // 16-byte vectors per thread and K step
  static_assert(TM % 32 == 0 && TN % 32 == 0 && VA >= 1 && VB >= 1, "tile shape");
  __shared__ __align__(16) uint16_t sAll[(2 * BM + BN) * GB_PITCH];     // one block: the GU epilogue reuses it
  uint16_t* sAh = sAll;
  uint16_t* sAl = sAll + BM * GB_PITCH;
  uint16_t* sB = sAll + 2 * BM * GB_PITCH;
  static_assert(!GU || (WGN == 2 && VB % 2 == 0 && (size_t)BM * (BN / 2) * 4 <= sizeof(sAll)), "gate columns | up columns");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = (wave / WGN) * TM, wn = (wave % WGN) * TN;
  floatx16_t acc[IM][JN];
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // Two K steps of operands are in flight in registers: a load takes longer than the matrix cores need for one step.
  // The loads are issued through inline asm and waited for by count (the compiler would sink ordinary loads down to
  // their first use and wait for all of them at every barrier): rows and K offsets past the end are clamped for the
  // load and zeroed when the registers go to LDS, the step count is rounded up to a multiple of the stages, the barriers wait for LDS
  // only, and pf_wait<NL> lets exactly the other stage's NL loads stay outstanding (loads return in order).
  struct Stage { u32x4_t h[VA], l[VA], b[VB]; };
  constexpr int NL = 2 * VA + VB;
  const int nsteps = (K + GB_K - 1) / GB_K;
  auto fetch = [&](Stage& R, int step) __attribute__((always_inline)) {
    const int k0 = min(step, nsteps - 1) * GB_K;
#pragma unroll
    for (int i = 0; i < VA; ++i) {
      const int v = tid + WG * i, row = min(m0 + (v >> 3), M - 1), k = min(k0 + ((v & 7) << 3), K - 8);
      pf_issue16(R.h[i], Ah + (size_t)row * K + k);
      pf_issue16(R.l[i], Al + (size_t)row * K + k);
    }
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int v = tid + WG * i, k = min(k0 + ((v & 7) << 3), K - 8);
      if (GU) {                                        // rows 0 .. BN/2-1 of the tile: gate, the rest: up (i decides)
        const int row = min(n0 + ((v >> 3) & (BN / 2 - 1)), N - 1);
        pf_issue16(R.b[i], (i < VB / 2 ? W : W2) + (size_t)row * K + k);
      } else {
        const int row = min(n0 + (v >> 3), N - 1);
        pf_issue16(R.b[i], W + (size_t)row * K + k);
      }
    }
  };
  auto stash = [&](Stage& R, int step) __attribute__((always_inline)) {
    const int k0 = step * GB_K;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < VA; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      const bool ok = step < nsteps && k0 + kc < K && m0 + row < M;
      pf_use(R.h[i]); pf_use(R.l[i]);
      *reinterpret_cast<u32x4_t*>(sAh + row * GB_PITCH + kc) = ok ? R.h[i] : zero;
      *reinterpret_cast<u32x4_t*>(sAl + row * GB_PITCH + kc) = ok ? R.l[i] : zero;
    }
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int v = tid + WG * i, row = v >> 3, kc = (v & 7) << 3;
      const bool ok = step < nsteps && k0 + kc < K && n0 + (GU ? (row & (BN / 2 - 1)) : row) < N;
      pf_use(R.b[i]);
      *reinterpret_cast<u32x4_t*>(sB + row * GB_PITCH + kc) = ok ? R.b[i] : zero;
    }
  };
  auto compute = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < GB_K; kk += 16) {
      bf16x8_t ah[IM], al[IM], b[JN];
#pragma unroll
      for (int i = 0; i < IM; ++i) {
        const int ao = (wm + i * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3);
        ah[i] = *reinterpret_cast<const bf16x8_t*>(sAh + ao);
        al[i] = *reinterpret_cast<const bf16x8_t*>(sAl + ao);
      }
#pragma unroll
      for (int j = 0; j < JN; ++j)
        b[j] = *reinterpret_cast<const bf16x8_t*>(sB + (wn + j * 32 + (lane & 31)) * GB_PITCH + kk + ((lane >> 5) << 3));
      // low halves first, then high halves: two products into the same accumulator are never issued back to back
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[i], b[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[i], b[j], acc[i][j], 0, 0, 0);
    }
  };

  // NSTG stages (K steps) of operands in flight; the loop is unrolled over the stages so that every stage is a fixed
  // set of registers.
  Stage R[NSTG];
#pragma unroll
  for (int q = 0; q < NSTG; ++q) fetch(R[q], q);
  for (int s = 0; s < nsteps; s += NSTG) {
#pragma unroll
    for (int q = 0; q < NSTG; ++q) {
      lds_barrier();                       // everyone has read the previous step's tiles
      pf_wait<NL * (NSTG - 1)>();          // this stage has landed; the younger ones may still be on their way
      stash(R[q], s + q);
      lds_barrier();
      fetch(R[q], s + q + NSTG);
      compute();
    }
  }
  // The last fetches (clamped re-loads nobody reads) are still on their way: wait for them, and only then let go of
  // their destinations - the compiler would otherwise hand those registers to the epilogue's addresses while the loads
  // can still land in them.
  pf_wait<0>();
#pragma unroll
  for (int q = 0; q < NSTG; ++q) {
#pragma unroll
    for (int i = 0; i < VA; ++i) { pf_use(R[q].h[i]); pf_use(R[q].l[i]); }
#pragma unroll
    for (int i = 0; i < VB; ++i) pf_use(R[q].b[i]);
  }
  if constexpr (GU) {
    // the up waves (wn != 0) pass their accumulators through LDS to the gate waves of the same rows
    float* u_lds = reinterpret_cast<float*>(sAll);                 // [BM][BN / 2]
    lds_barrier();                                                 // every wave has finished reading the operand tiles
    if (wn != 0) {
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            u_lds[(wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * (BN / 2) + j * 32 + (lane & 31)] = acc[i][j][r];
    }
    lds_barrier();
    if (wn == 0) {
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const int col = n0 + j * 32 + (lane & 31);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int rl = wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), row = m0 + rl;
            if (row < M && col < N) {
              const float z = siluf(acc[i][j][r]) * u_lds[rl * (BN / 2) + j * 32 + (lane & 31)];
              const bf16 h = from_f32<bf16>(z);
              zh[(size_t)row * N + col] = h;
              zl[(size_t)row * N + col] = from_f32<bf16>(z - to_f32(h));
            }
          }
        }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < IM; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const int col = n0 + wn + j * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + wm + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row < M && col < N) {
          float* c = C + (size_t)row * N + col;
          *c = accumulate ? *c + acc[i][j][r] : acc[i][j][r];
        }
      }
    }
}

// Several weight matrices applied to the same activations in one launch (Q, K and V; gate and up): the column
// blocks of the segments follow each other in blockIdx.x, each segment with its own matrix, output and width.
// A matrix of 1024 rows alone is 64 workgroups at 1024 tokens - a quarter of the compute units; together the
// projections of one input fill whole rounds.
struct GemmSeg { const bf16* W; float* C; int N; int blocks; };     // blocks = ceil(N / GB_N)
struct GemmSegs { GemmSeg s[3]; int n; };
__global__ void __launch_bounds__(WG) k_gemm_nt_bf16_hl_seg(const bf16* __restrict__ Ah, const bf16* __restrict__ Al,
                                                            GemmSegs segs, int M, int K, int accumulate) {
  int bx = blockIdx.x, i = 0;
  while (i + 1 < segs.n && bx >= segs.s[i].blocks) { bx -= segs.s[i].blocks; ++i; }
  const GemmSeg g = segs.s[i];
  gemm_nt_bf16_hl_tile<GB_M, GB_N, 2, 2>(Ah, Al, g.W, g.C, M, g.N, K, accumulate, blockIdx.y * GB_M, bx * GB_N);
}
// The same with 64-row tiles, for shapes whose 128 x 128 tiles would leave every compute unit a single workgroup
// (one wave per SIMD, nothing to overlap a barrier or a load with): twice the workgroups, two per compute unit.  Four layers of
// the 8B shape with every matrix off 16 bytes, 128 / 512 / 1000 rows: 2.73 / 3.75 / 5.05 ms without, 2.07 / 2.98 / 4.96 with.
constexpr int GB_MS = 64;
__global__ void __launch_bounds__(WG) k_gemm_nt_bf16_hl_seg_s(const bf16* __restrict__ Ah, const bf16* __restrict__ Al,
                                                              GemmSegs segs, int M, int K, int accumulate) {
  int bx = blockIdx.x, i = 0;
  while (i + 1 < segs.n && bx >= segs.s[i].blocks) { bx -= segs.s[i].blocks; ++i; }
  const GemmSeg g = segs.s[i];
  gemm_nt_bf16_hl_tile<GB_MS, GB_N, 2, 2>(Ah, Al, g.W, g.C, M, g.N, K, accumulate, blockIdx.y * GB_MS, bx * GB_N);
}

// Gate and up projections with SiLU(gate) * up in the epilogue: a workgroup takes 64 columns of both matrices for its
// 128 rows, so the MLP activation leaves the GEMM already split for the down projection - no fp32 gate / up
// matrices in memory and no elementwise launch.  N = d_ffn.
__global__ void __launch_bounds__(WG) k_gemm_nt_bf16_hl_gu(const bf16* __restrict__ Ah, const bf16* __restrict__ Al,
                                                           const bf16* __restrict__ Wg, const bf16* __restrict__ Wu,
                                                           bf16* __restrict__ zh, bf16* __restrict__ zl, int M, int N, int K) {
  gemm_nt_bf16_hl_tile<GB_M, GB_N, 2, 2, 2, true>(Ah, Al, Wg, nullptr, M, N, K, 0, blockIdx.y * GB_M, blockIdx.x * (GB_N / 2), Wu,
                                                  zh, zl);
}

// fp32 variant (the small full-precision configuration): 64x64 tile, 4x4 per thread.
__global__ void __launch_bounds__(WG) k_gemm_nt_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                    float* __restrict__ C, int M, int N, int K, int accumulate) {
  __shared__ __align__(16) float sA[16][68];
  __shared__ __align__(16) float sB[16][68];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int lr = tid >> 2, lk = (tid & 3) << 2;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    float4 va = make_float4(0, 0, 0, 0), vb = make_float4(0, 0, 0, 0);
    if (k0 + lk < K) {
      if (m0 + lr < M) va = *reinterpret_cast<const float4*>(A + (size_t)(m0 + lr) * K + k0 + lk);
      if (n0 + lr < N) vb = *reinterpret_cast<const float4*>(W + (size_t)(n0 + lr) * K + k0 + lk);
    }
    __syncthreads();
    sA[lk][lr] = va.x; sA[lk + 1][lr] = va.y; sA[lk + 2][lr] = va.z; sA[lk + 3][lr] = va.w;
    sB[lk][lr] = vb.x; sB[lk + 1][lr] = vb.y; sB[lk + 2][lr] = vb.z; sB[lk + 3][lr] = vb.w;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float4 a = *reinterpret_cast<const float4*>(&sA[k][ty * 4]);
      const float4 b = *reinterpret_cast<const float4*>(&sB[k][tx * 4]);
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = m0 + ty * 4 + i, col = n0 + tx * 4 + j;
      if (row < M && col < N) {
        float* c = C + (size_t)row * N + col;
        *c = accumulate ? *c + acc[i][j] : acc[i][j];
      }
    }
}

// The same for shapes whose 64 x 64 tiles would leave most of the chip idle (short prompts of a small model): S TT x S TT
// tiles, S x S threads, TT x TT outputs per thread, K in steps of 256 / TT with the next step already on its way in registers.  Up to three matrices
// applied to the same rows, their column tiles one after the other; GU: matrix 0 is the gate, 1 up, and C[0] = SiLU(gate) * up.  Every
// output is the same chain of multiply-adds over ascending k, so the bits are those of k_gemm_nt_f32 (and k_silu_mul).  Bound: latency, a
// memory round trip per step (32 x 256 x 256: 17.6 us in 64 x 64 tiles, 5.8 in steps of 64, 5.2 now - Q, K and V together 5.2 -;
// 32 x 256 x 688: 49.4, 14.0, 10.1; gate and up of 32 x 688 x 256 with SiLU 6.0 + 6.0 + 2.1 in three launches, 7.0 here; kernel trace).  With one
// output a thread a multiply-add waits for 8 bytes from LDS: 16 x 16 tiles that leave half the chip without one are cut into four
// (32 tokens, four layers of 256 x 688: 267 us a prompt pass, 245 so).
struct SmallSegs { const float* W[3]; float* C[3]; int N[3], blocks[3]; };
template <int S, int TT, bool GU>
__global__ void __launch_bounds__(S * S) k_gemm_nt_f32_small(const float* __restrict__ A, SmallSegs segs, int M, int K, int accumulate) {
  constexpr int N_THR = S * S, T = S * TT, BK = 256 / TT, PITCH = BK + 4, NB = GU ? 2 : 1;      // (rows 16 bytes apart modulo the banks)
  constexpr int PR = BK / 4, NP = T * PR / N_THR;             // pieces of 16 bytes in a row of a step; pieces of a thread
  __shared__ __align__(16) float sA[T * PITCH], sB[NB][T * PITCH];
  int bx = blockIdx.x, si = 0;
  if (!GU)
    while (si < 2 && bx >= segs.blocks[si]) bx -= segs.blocks[si++];
  const float* const W = segs.W[si];
  float* const C = segs.C[si];
  const int N = segs.N[si];
  const int tid = threadIdx.x, tx = tid & (S - 1), ty = tid / S, m0 = blockIdx.y * T, n0 = bx * T;
  float4 ra[NP], rb[NB][NP];
  auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int row = (u * N_THR + tid) / PR, k = k0 + (u * N_THR + tid) % PR * 4;
      // (a piece that exists is loaded whatever happens and zeroed afterwards: choosing between a load and a constant makes
      // the compiler choose between two addresses, one of them in scratch memory)
      ra[u] = keep4(*reinterpret_cast<const float4*>(A + (size_t)min(m0 + row, M - 1) * K + min(k, K - 4)), k < K && m0 + row < M);
#pragma unroll
      for (int b = 0; b < NB; ++b)
        rb[b][u] = keep4(*reinterpret_cast<const float4*>((b ? segs.W[1] : W) + (size_t)min(n0 + row, N - 1) * K + min(k, K - 4)), k < K && n0 + row < N);
    }
  };
  float acc[NB][TT][TT] = {};
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NP; ++u) {
      const int at = (u * N_THR + tid) / PR * PITCH + (u * N_THR + tid) % PR * 4;
      *reinterpret_cast<float4*>(sA + at) = ra[u];
#pragma unroll
      for (int b = 0; b < NB; ++b) *reinterpret_cast<float4*>(sB[b] + at) = rb[b][u];
    }
    __syncthreads();
    if (k0 + BK < K) fetch(k0 + BK);
    const int kn = min(BK, K - k0);                        // a multiple of 4: K is one of 8
#pragma unroll 8
    for (int k = 0; k < kn; k += 4) {
      float4 a[TT], w[NB][TT];
#pragma unroll
      for (int u = 0; u < TT; ++u) {
        a[u] = *reinterpret_cast<const float4*>(sA + (u * S + ty) * PITCH + k);
#pragma unroll
        for (int b = 0; b < NB; ++b) w[b][u] = *reinterpret_cast<const float4*>(sB[b] + (u * S + tx) * PITCH + k);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < TT; ++i)
#pragma unroll
          for (int j = 0; j < TT; ++j) {
            float& t = acc[b][i][j];
            t = fmaf(a[i].x, w[b][j].x, t); t = fmaf(a[i].y, w[b][j].y, t);
            t = fmaf(a[i].z, w[b][j].z, t); t = fmaf(a[i].w, w[b][j].w, t);
          }
    }
  }
#pragma unroll
  for (int i = 0; i < TT; ++i)
#pragma unroll
    for (int j = 0; j < TT; ++j) {
      const int row = m0 + i * S + ty, col = n0 + j * S + tx;
      if (row < M && col < N) {
        float* c = C + (size_t)row * N + col;
        if (GU) *c = siluf(acc[0][i][j]) * acc[NB - 1][i][j];
        else *c = accumulate ? *c + acc[0][i][j] : acc[0][i][j];
      }
    }
}

// ---------------------------------------------------------------------------------------
// Per token: rotate q (in place, pre-scaled by 1/sqrt(hd)), rotate k, round k and v to the
// cache type and write them to the token's page slot.  grid = rows of the group.
template <typename KVT>
__global__ void __launch_bounds__(WG) k_rope_kvwrite(float* __restrict__ q, const float* __restrict__ kraw,
                                                     const float* __restrict__ vraw, const float2* __restrict__ cs,
                                                     PromptPack pk, KVT* __restrict__ pool,
                                                     size_t page_elems, int Hq, int Hkv, int hd, int P, float qscale) {
  const int r = blockIdx.x, half = hd >> 1, j = pack_find(pk.off, pk.n, r), t = r - (pk.off[j] - pk.off[0]);
  const int* pt = pk.pt + (size_t)(pk.b0 + j) * pk.max_pages;
  const float2* c = cs + (size_t)t * half;
  float* qrow = q + (size_t)r * Hq * hd;
  for (int i = threadIdx.x; i < Hq * half; i += WG) {
    const int h = i / half, d = i - h * half;
    const float x1 = qrow[h * hd + d], x2 = qrow[h * hd + d + half];
    qrow[h * hd + d] = (x1 * c[d].x - x2 * c[d].y) * qscale;
    qrow[h * hd + d + half] = (x2 * c[d].x + x1 * c[d].y) * qscale;
  }
  const size_t base = (size_t)pt[t / P] * page_elems + (size_t)(t % P) * hd;
  const size_t v_off = (size_t)Hkv * P * hd;
  const float* krow = kraw + (size_t)r * Hkv * hd;
  const float* vrow = vraw + (size_t)r * Hkv * hd;
  for (int i = threadIdx.x; i < Hkv * half; i += WG) {
    const int g = i / half, d = i - g * half;
    const float x1 = krow[g * hd + d], x2 = krow[g * hd + d + half];
    KVT* dst = pool + base + (size_t)g * P * hd;
    dst[d] = from_f32<KVT>(x1 * c[d].x - x2 * c[d].y);
    dst[d + half] = from_f32<KVT>(x2 * c[d].x + x1 * c[d].y);
  }
  for (int i = threadIdx.x; i < Hkv * hd; i += WG) {
    const int g = i / hd, d = i - g * hd;
    pool[base + v_off + (size_t)g * P * hd + d] = from_f32<KVT>(vrow[i]);
  }
}

// Causal GQA attention over the prompt, reading K and V back from the cache pages.
// grid = (ceil(T/QB), Hkv); the workgroup owns QB query positions x G heads (<= 64 rows),
// one wave per row in turn; 64-key tiles of K (padded rows) and V are shared through LDS.
// Bound: the chain of one row - 64 multiply-adds of a score, a value a key -, so what it reads from LDS is requested eight at a time (prompts of an fp32 model of
// four layers, 256 x 688, us a pass before / after: 200 tokens 384 / 348, 1000 1387 / 1094, 2000 4088 / 2920; the same sums in the same order).
constexpr int PA_RPW = 16;      // rows per wave
template <typename XT, typename KVT>
__global__ void __launch_bounds__(WG) k_attn_prefill(const float* __restrict__ q, XT* __restrict__ out,
                                                     const int* __restrict__ pt, const KVT* __restrict__ pool,
                                                     size_t page_elems, int T, int Hq, int Hkv, int hd, int P, int QB) {
  extern __shared__ __align__(16) float smem_f[];
  constexpr int VEC = Vec<KVT>::N;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int G = Hq / Hkv, g = blockIdx.y, t0 = blockIdx.x * QB;
  const int NR = QB * G;
  float* qs = smem_f;                                              // [NR][hd]
  char* kt = reinterpret_cast<char*>(qs + 64 * hd);
  const int kpitch = hd * (int)sizeof(KVT) + 4;
  const KVT* vt = reinterpret_cast<const KVT*>(kt + 64 * kpitch);
  KVT* vtw = reinterpret_cast<KVT*>(kt + 64 * kpitch);
  const size_t head_off = (size_t)g * P * hd, v_off = (size_t)Hkv * P * hd;

  for (int i = tid; i < NR * hd; i += WG) {
    const int rr = i / hd, d = i - rr * hd;
    const int t = t0 + rr / G, H = g * G + rr % G;
    qs[i] = (t < T) ? q[((size_t)t * Hq + H) * hd + d] : 0.f;
  }
  float m[PA_RPW], l[PA_RPW], o0[PA_RPW], o1[PA_RPW];
#pragma unroll
  for (int i = 0; i < PA_RPW; ++i) { m[i] = -INFINITY; l[i] = 0.f; o0[i] = 0.f; o1[i] = 0.f; }

  const int k_end = min(T, t0 + QB);
  const int vec_per_key = hd / VEC;
  for (int kt0 = 0; kt0 < k_end; kt0 += 64) {
    __syncthreads();
    for (int i = tid; i < 64 * vec_per_key; i += WG) {
      const int j = i / vec_per_key, c = (i - j * vec_per_key) * VEC;
      const int key = kt0 + j;
      uint4 kv4 = make_uint4(0, 0, 0, 0), vv4 = make_uint4(0, 0, 0, 0);
      if (key < k_end) {
        const size_t base = (size_t)pt[key / P] * page_elems + head_off + (size_t)(key % P) * hd + c;
        kv4 = *reinterpret_cast<const uint4*>(pool + base);
        vv4 = *reinterpret_cast<const uint4*>(pool + base + v_off);
      }
      uint32_t* kd = reinterpret_cast<uint32_t*>(kt + j * kpitch + c * sizeof(KVT));
      kd[0] = kv4.x; kd[1] = kv4.y; kd[2] = kv4.z; kd[3] = kv4.w;
      *reinterpret_cast<uint4*>(vtw + j * hd + c) = vv4;
    }
    __syncthreads();
#pragma unroll
    for (int ri = 0; ri < PA_RPW; ++ri) {
      const int rr = wave + ri * WAVES;
      const int t = t0 + rr / G;
      if (rr < NR && t < T && kt0 <= t) {
        const int jn = min(64, t - kt0 + 1);
        float sc = 0.f;
        const char* krow = kt + lane * kpitch;
        const float* qv = qs + rr * hd;
        if (sizeof(KVT) == 2) {
#pragma unroll 16
          for (int d = 0; d < hd; d += 2) {
            const uint32_t w2 = *reinterpret_cast<const uint32_t*>(krow + d * 2);
            sc = fmaf(qv[d], __uint_as_float(w2 << 16), sc);
            sc = fmaf(qv[d + 1], __uint_as_float(w2 & 0xffff0000u), sc);
          }
        } else {
#pragma unroll 4
          for (int d = 0; d < hd; d += 8) {                // (hd: a multiple of 8)
            float k8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) k8[e] = *reinterpret_cast<const float*>(krow + (d + e) * 4);
            const float4 qa = *reinterpret_cast<const float4*>(qv + d), qb = *reinterpret_cast<const float4*>(qv + d + 4);
            sc = fmaf(qa.x, k8[0], sc); sc = fmaf(qa.y, k8[1], sc); sc = fmaf(qa.z, k8[2], sc); sc = fmaf(qa.w, k8[3], sc);
            sc = fmaf(qb.x, k8[4], sc); sc = fmaf(qb.y, k8[5], sc); sc = fmaf(qb.z, k8[6], sc); sc = fmaf(qb.w, k8[7], sc);
          }
        }
        if (lane >= jn) sc = -INFINITY;
        const float mn = fmaxf(m[ri], wave_max(sc));
        const float corr = expf(m[ri] - mn);
        const float pj = (lane < jn) ? expf(sc - mn) : 0.f;
        l[ri] = l[ri] * corr + wave_sum(pj);
        o0[ri] *= corr; o1[ri] *= corr;
        m[ri] = mn;
        // eight values requested together (one at a time each waited for LDS: 32 keys of a row 1.8 us); behind the row's own position weight and value are zero
        const int c0 = min(lane, hd - 1), c1 = min(lane + 64, hd - 1);
        for (int j0 = 0; j0 < jn; j0 += 8) {
          KVT v0[8], v1[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            v0[u] = vt[(j0 + u) * hd + c0];
            if (hd > 64) v1[u] = vt[(j0 + u) * hd + c1];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const float pb = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pj), j0 + u));
            o0[ri] = fmaf(pb, j0 + u < jn ? to_f32(v0[u]) : 0.f, o0[ri]);
            if (hd > 64) o1[ri] = fmaf(pb, j0 + u < jn ? to_f32(v1[u]) : 0.f, o1[ri]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int ri = 0; ri < PA_RPW; ++ri) {
    const int rr = wave + ri * WAVES;
    const int t = t0 + rr / G, H = g * G + rr % G;
    if (rr < NR && t < T) {
      XT* o = out + ((size_t)t * Hq + H) * hd;
      if (lane < hd) o[lane] = from_f32<XT>(o0[ri] / l[ri]);
      if (lane + 64 < hd) o[lane + 64] = from_f32<XT>(o1[ri] / l[ri]);
    }
  }
}

// z = silu(g) * u in the GEMM input type.
template <typename XT>
__global__ void __launch_bounds__(WG) k_silu_mul(const float* __restrict__ g, const float* __restrict__ u,
                                                 XT* __restrict__ z, size_t n) {
  for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n; i += (size_t)gridDim.x * WG)
    z[i] = from_f32<XT>(siluf(g[i]) * u[i]);
}

// fp32 -> hi / lo bf16.  grid-stride over n elements.
__global__ void __launch_bounds__(WG) k_split_bf16(const float* __restrict__ x, bf16* __restrict__ hi, bf16* __restrict__ lo, size_t n) {
  for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n; i += (size_t)gridDim.x * WG) {
    const float v = x[i];
    const bf16 h = from_f32<bf16>(v);
    hi[i] = h;
    lo[i] = from_f32<bf16>(v - to_f32(h));
  }
}

__global__ void k_set_int(int* p, int v) { if (threadIdx.x == 0 && blockIdx.x == 0) *p = v; }

// KV taps: positions [pos0, pos0+n) of one layer <-> dense fp32 [n][Hkv][hd].
template <typename KVT, bool WRITE>
__global__ void __launch_bounds__(WG) k_kv_tap(KVT* __restrict__ pool, size_t page_elems, const int* __restrict__ pt,
                                               int pos0, int Hkv, int hd, int P, float* __restrict__ kbuf,
                                               float* __restrict__ vbuf) {
  const int j = blockIdx.x, pos = pos0 + j;
  const size_t base = (size_t)pt[pos / P] * page_elems + (size_t)(pos % P) * hd;
  const size_t v_off = (size_t)Hkv * P * hd;
  for (int i = threadIdx.x; i < Hkv * hd; i += WG) {
    const int g = i / hd, d = i - g * hd;
    const size_t a = base + (size_t)g * P * hd + d;
    if (WRITE) {
      pool[a] = from_f32<KVT>(kbuf[(size_t)j * Hkv * hd + i]);
      pool[a + v_off] = from_f32<KVT>(vbuf[(size_t)j * Hkv * hd + i]);
    } else {
      kbuf[(size_t)j * Hkv * hd + i] = to_f32(pool[a]);
      vbuf[(size_t)j * Hkv * hd + i] = to_f32(pool[a + v_off]);
    }
  }
}

}  // namespace first
