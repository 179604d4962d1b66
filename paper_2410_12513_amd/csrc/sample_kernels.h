// Temperature + top-k sampling over the logits of a decode step (Appendix, "Inference
// settings": temperature 0.8, top-k sampling over 10 tokens).  The draw itself is a uniform
// number in [0, 1) supplied by the caller, one per sequence: the library owns no random
// number generator.
//
//   candidates = the k largest logits, equal logits ordered by token index (lowest first);
//   p_j ~ exp((l_j - l_max) / T) over the candidates, summed in descending-logit order;
//   result = the first candidate whose cumulative weight exceeds u * total.
//
// Two stages: every wave of k_topk_part selects the top k of its 512 logits (k rounds of "the largest key left", keys in
// registers, no barrier), the workgroup merges its four lists by rank; k_topk_sample does the same with the lists of one
// sequence and draws.  All fp32, fixed order.
#pragma once
#include "common.h"

namespace first {

constexpr int SMP_THREADS = 256;
constexpr int SMP_VPT = 8;                              // logits per thread in stage 1
constexpr int SMP_CHUNK = SMP_THREADS * SMP_VPT;
constexpr int SMP_KMAX = 64;
constexpr int SMP_NONE = 0x7fffffff;                    // index of "no candidate"

struct Cand { float v; int i; };

// a comes before b: larger logit, or equal logit and lower index
__device__ __forceinline__ bool cand_before(const Cand& a, const Cand& b) {
  return a.v > b.v || (a.v == b.v && a.i < b.i);
}

// The order as an unsigned key: a comes before b iff key(a) > key(b).  Upper word: the logit's bits in ascending order (-0 counts
// as 0), lower word: ~index.  0: no candidate (a NaN is none either).
__device__ __forceinline__ unsigned long long cand_key(float v, int i) {
  const uint32_t u = __float_as_uint(v + 0.f);
  const uint32_t o = (u & 0x80000000u) ? ~u : u | 0x80000000u;
  return i == SMP_NONE || v != v ? 0ull : ((unsigned long long)o << 32) | (uint32_t)~i;
}
__device__ __forceinline__ Cand cand_of(unsigned long long key) {
  const uint32_t o = (uint32_t)(key >> 32);
  return key == 0ull ? Cand{-INFINITY, SMP_NONE} : Cand{__uint_as_float((o & 0x80000000u) ? o & 0x7fffffffu : ~o), (int)~(uint32_t)key};
}
// Largest value over the wave (DPP: quads, half rows, rows, then the two row broadcasts of gfx9), in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define FIRST_DPP_MAX(CTRL, ROWS) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false))
  FIRST_DPP_MAX(0xB1, 0xf); FIRST_DPP_MAX(0x4E, 0xf); FIRST_DPP_MAX(0x141, 0xf); FIRST_DPP_MAX(0x140, 0xf);
  FIRST_DPP_MAX(0x142, 0xa); FIRST_DPP_MAX(0x143, 0xc);
#undef FIRST_DPP_MAX
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// list[0 .. k) = the k largest of the wave's keys, in order (0 behind the last one).  Takes them out of e.
__device__ __forceinline__ void wave_top(unsigned long long (&e)[SMP_VPT], int k, unsigned long long* list) {
  for (int r = 0; r < k; ++r) {
    unsigned long long best = e[0];
#pragma unroll
    for (int j = 1; j < SMP_VPT; ++j) best = e[j] > best ? e[j] : best;
    const uint32_t hi = wave_max_u32((uint32_t)(best >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(best >> 32) == hi ? (uint32_t)best : 0u);
    const unsigned long long first = ((unsigned long long)hi << 32) | lo;
#pragma unroll
    for (int j = 0; j < SMP_VPT; ++j)
      if (e[j] == first) e[j] = 0ull;
    if ((threadIdx.x & 63) == 0) list[r] = first;
  }
}
// top[0 .. k) = the k largest of the n keys (all different but for the zeros): a key's place is the number of larger ones.
__device__ __forceinline__ void rank_merge(const unsigned long long* keys, int n, int k, unsigned long long* top) {
  if ((int)threadIdx.x < k) top[threadIdx.x] = 0ull;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += SMP_THREADS) {
    const unsigned long long x = keys[i];
    int before = 0;
    for (int j = 0; j < n; ++j) before += keys[j] > x;
    if (x != 0ull && before < k) top[before] = x;
  }
  __syncthreads();
}

// The draw: top[0..k) in order (SMP_NONE beyond the vocabulary), u in [0, 1).  One thread.  smp_draw forms the weights as it
// goes (the persistent kernel's single lane), smp_pick takes them ready (formed side by side by the lanes of
// k_topk_sample): the same values, the same sums, the same decision.
__device__ __forceinline__ float smp_weight(const Cand& c, const Cand& best, float temperature) { return expf((c.v - best.v) / temperature); }
__device__ __forceinline__ int smp_draw(const Cand* top, int k, float temperature, float u) {
  int kk = 0;
  while (kk < k && top[kk].i != SMP_NONE) ++kk;
  const float lmax = top[0].v;
  float total = 0.f;
  for (int j = 0; j < kk; ++j) total += expf((top[j].v - lmax) / temperature);
  const float target = u * total;
  float cum = 0.f;
  int pick = kk > 0 ? top[kk - 1].i : 0;
  for (int j = 0; j < kk; ++j) {
    cum += expf((top[j].v - lmax) / temperature);
    if (cum > target) { pick = top[j].i; break; }
  }
  return pick;
}
__device__ __forceinline__ int smp_pick(const Cand* top, const float* weight, int k, float u) {
  int kk = 0;
  while (kk < k && top[kk].i != SMP_NONE) ++kk;
  float total = 0.f;
  for (int j = 0; j < kk; ++j) total += weight[j];
  const float target = u * total;
  float cum = 0.f;
  int pick = kk > 0 ? top[kk - 1].i : 0;
  for (int j = 0; j < kk; ++j) {
    cum += weight[j];
    if (cum > target) { pick = top[j].i; break; }
  }
  return pick;
}

// Stage 1.  grid (chunks, sequences).  part[(seq * chunks + chunk) * k + r] = r-th candidate of the chunk.
// Latency, not bandwidth (16 x 128256 logits, k = 10, kernel trace: 23.3 us with a barrier pair and an LDS reduction per
// candidate, 10.5 now; 8 MB).
__global__ void __launch_bounds__(SMP_THREADS) k_topk_part(const float* __restrict__ logits, int V, int k, Cand* __restrict__ part) {
  __shared__ unsigned long long lists[(SMP_THREADS / 64) * SMP_KMAX], top[SMP_KMAX];
  const int tid = threadIdx.x, chunk = blockIdx.x, seq = blockIdx.y;
  const float* row = logits + (size_t)seq * V;
  float v[SMP_VPT];
#pragma unroll
  for (int j = 0; j < SMP_VPT; ++j) v[j] = row[min(chunk * SMP_CHUNK + j * SMP_THREADS + tid, V - 1)];
  unsigned long long e[SMP_VPT];
#pragma unroll
  for (int j = 0; j < SMP_VPT; ++j) {
    const int idx = chunk * SMP_CHUNK + j * SMP_THREADS + tid;
    e[j] = idx < V ? cand_key(v[j], idx) : 0ull;
  }
  wave_top(e, k, lists + (tid >> 6) * k);
  rank_merge(lists, (SMP_THREADS / 64) * k, k, top);       // (begins with a barrier)
  if (tid < k) part[((size_t)seq * gridDim.x + chunk) * k + tid] = cand_of(top[tid]);
}

// Stage 2.  grid (sequences).  n = chunks * k candidates of the sequence, 2048 at a time (17.2 us before at n = 630, 10.1 now).
__global__ void __launch_bounds__(SMP_THREADS) k_topk_sample(const Cand* __restrict__ part, int n, int k, float temperature,
                                                            const float* __restrict__ uniforms, int* __restrict__ token_out,
                                                            int* __restrict__ cand_out) {
  __shared__ unsigned long long lists[(SMP_THREADS / 64 + 1) * SMP_KMAX], top[SMP_KMAX];
  __shared__ Cand first[SMP_KMAX];
  __shared__ float weight[SMP_KMAX];
  const int tid = threadIdx.x, seq = blockIdx.x;
  const Cand* c = part + (size_t)seq * n;
  const float u = uniforms[seq];
  if (tid < k) top[tid] = 0ull;
  for (int base = 0; base < n; base += SMP_CHUNK) {
    unsigned long long e[SMP_VPT];
#pragma unroll
    for (int j = 0; j < SMP_VPT; ++j) {
      const int at = base + j * SMP_THREADS + tid;
      const Cand x = c[min(at, n - 1)];
      e[j] = at < n ? cand_key(x.v, x.i) : 0ull;
    }
    wave_top(e, k, lists + (tid >> 6) * k);
    if (tid < k) lists[(SMP_THREADS / 64) * k + tid] = top[tid];          // what the candidates before these came to
    __syncthreads();
    rank_merge(lists, (SMP_THREADS / 64 + 1) * k, k, top);
  }
  if (tid < k) {
    const Cand t = cand_of(top[tid]);
    first[tid] = t;
    weight[tid] = smp_weight(t, cand_of(top[0]), temperature);           // (side by side; one thread adds them up)
    if (cand_out != nullptr) cand_out[(size_t)seq * k + tid] = t.i == SMP_NONE ? -1 : t.i;
  }
  __syncthreads();
  if (tid == 0) token_out[seq] = smp_pick(first, weight, k, u);
}

}  // namespace first
