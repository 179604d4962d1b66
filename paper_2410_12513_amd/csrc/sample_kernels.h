// Temperature + top-k sampling over the logits of a decode step (Appendix, "Inference
// settings": temperature 0.8, top-k sampling over 10 tokens).  The draw itself is a uniform
// number in [0, 1) supplied by the caller, one per sequence: the library owns no random
// number generator.
//
//   candidates = the k largest logits, equal logits ordered by token index (lowest first);
//   p_j ~ exp((l_j - l_max) / T) over the candidates, summed in descending-logit order;
//   result = the first candidate whose cumulative weight exceeds u * total.
//
// One workgroup a row; rows that are long for one compute unit in two stages: workgroups list the first k of 16384 logits or more each,
// a second launch merges the lists of a row and draws.  All fp32, fixed order.
#pragma once
#include "common.h"

namespace first {

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
// The draw: top[0..k) in order (SMP_NONE beyond the vocabulary), u in [0, 1).  smp_draw forms the weights as it goes (the
// persistent kernel's single lane), smp_draw_wave in the lanes of a wave: the same values, the same sums, the same decision.
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
__device__ __forceinline__ void smp_draw_wave(const unsigned long long* top, int k, float temperature, float u, int* token_out, int* cand_out) {
  const int lane = threadIdx.x & 63;
  const Cand c = cand_of(lane < k ? top[lane] : 0ull);
  const float w = smp_weight(c, cand_of(top[0]), temperature);
  if (lane < k && cand_out != nullptr) cand_out[lane] = c.i == SMP_NONE ? -1 : c.i;
  const int kk = __popcll(__ballot(c.i != SMP_NONE));
  auto weight = [&](int j) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(w), j)); };
  float total = 0.f;
  for (int j = 0; j < kk; ++j) total += weight(j);
  const float target = u * total;
  float cum = 0.f;
  int pick = kk > 0 ? kk - 1 : 0;
  for (int j = 0; j < kk; ++j) {
    cum += weight(j);
    if (cum > target) { pick = j; break; }
  }
  if (lane == pick) *token_out = kk > 0 ? c.i : 0;
}

// top[0 .. k) = the first k of the n keys (all different but for the zeros): a key's place is the number of larger ones.
__device__ __forceinline__ void rank_keys(const unsigned long long* keys, int n, int k, unsigned long long* top) {
  for (int i = threadIdx.x; i < n; i += (int)blockDim.x) {
    const unsigned long long x = keys[i];
    int before = 0, j = 0;
    for (; j + 8 <= n; j += 8)
#pragma unroll
      for (int e = 0; e < 8; ++e) before += keys[j + e] > x;
    for (; j < n; ++j) before += keys[j] > x;
    if (x != 0ull && before < k) top[before] = x;
  }
}

// What a draw asks before it writes behind the kernel of a whole decode step: whether a wait of that gave up (bit 0 of *err), so that its logits are none.  Other
// draws have no such argument.
struct DrawUnlessGivenUp {
  const int* err;
  __device__ __forceinline__ bool operator()() const { return (*err & 1) == 0; }
};

// The first k of a row (FINAL: and the draw; one launch, no scratch memory), or of part_len logits of it.  grid (parts, rows).
//
// First pass: a thread takes every 1024th piece of four logits (of one where they are few) and keeps the largest value and the LAST index of
// the piece it came from; a group of 16 lanes keeps the first of its threads in the sampling order.  The k-th of those 64 group
// maxima is a bound: at least k logits do not come behind it, and only threads whose own maximum does not can hold any of
// those - they alone read their logits a second time.  What they find, a dozen or two, is put in order by rank.  Ties are in the key, so
// masses of equal logits only make the list longer (64 k at most if all are equal).  A list that does not fit (logits where fewer than k groups
// have any that is not a NaN, or a pattern that puts the largest into a few groups) is replaced by k searches through all of them.
// Bound: latency, and what one compute unit reads (65 GB/s; 32000 logits 2 us).  k = 10, passes among others, 256 logits a wave in k
// rounds and two launches before: 16 rows of 128256 logits 10.9 us in two launches (6.5 + 4.2 in the kernel trace; 19.3), of 50257 10.1 in one
// (15.9), of 1024 6.2 (15.1).
constexpr int SMP_THREADS = 1024, SMP_LIST = 6144;
constexpr int SMP_PART = 16384;
constexpr int SMP_ROW_MAX = 65536;                       // longer rows in parts (16 rows of 65536, k = 10: 11.2 us in one launch, 10.1 in parts; 50257: 10.1)
struct __align__(4) Logits4 { float v[4]; };            // (a row starts on 4 bytes)

template <bool FINAL, typename... Draw>
__global__ void __launch_bounds__(SMP_THREADS) k_topk(const float* __restrict__ logits, int V, int part_len, int k, float temperature,
                                                     const float* __restrict__ uniforms, Cand* __restrict__ part,
                                                     int* __restrict__ token_out, int* __restrict__ cand_out, Draw... draw) {
  __shared__ __align__(16) unsigned long long list[SMP_LIST];
  __shared__ unsigned long long groups[64], top[SMP_KMAX], bound;
  __shared__ int found;
  constexpr int NW = SMP_THREADS / 64;                   // waves; lanes of a group: 64 groups
  static_assert(SMP_THREADS == 64 * 16, "groups are rows of 16 lanes");
  constexpr int U = FINAL ? 8 : 4;                       // pieces of a thread in flight (twice: the next ones while these are looked at)
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, seq = blockIdx.y;
  const int c0 = FINAL ? 0 : blockIdx.x * part_len, len = FINAL ? V : min(part_len, V - c0);
  const float* row = logits + (size_t)seq * V + c0;
  const float u = FINAL ? uniforms[seq] : 0.f;
  const int pieces = len < 4 * SMP_THREADS ? 0 : len / 4;
  const int mine = pieces > tid ? (pieces - tid + SMP_THREADS - 1) / SMP_THREADS : 0;
  auto fetch = [&](Logits4 (&x)[U], int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < U; ++j)                          // (past the end: a piece there is, not used)
      x[j] = *reinterpret_cast<const Logits4*>(row + 4 * (tid + SMP_THREADS * max(0, min(i + j, mine - 1))));
  };
  float m = -INFINITY;
  int last = SMP_NONE;
  auto take = [&](float v, int idx) __attribute__((always_inline)) {
    if (v > m || (last == SMP_NONE && v == v)) { m = v; last = idx; }
  };
  if (tid == 0) { bound = 0ull; found = 0; }
  if (tid < SMP_KMAX) top[tid] = 0ull;
  // logits that are in no piece of four: the last three at most, or all of them
  float single[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = pieces * 4 + tid + SMP_THREADS * j;
    single[j] = i < len ? row[i] : NAN;
  }
  if (mine > 0) {
    Logits4 a[U], b[U];
    auto look = [&](const Logits4 (&x)[U], int i) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < U; ++j)
        if (i + j < mine) take(fmaxf(fmaxf(x[j].v[0], x[j].v[1]), fmaxf(x[j].v[2], x[j].v[3])), 4 * (tid + SMP_THREADS * (i + j)) + 3);
    };
    fetch(a, 0);
    for (int i = 0; i < mine; i += 2 * U) {              // (requests only for pieces there are: repeated ones cost 1.5 us of a part's 5)
      if (i + U < mine) fetch(b, i + U);
      look(a, i);
      if (i + 2 * U < mine) fetch(a, i + 2 * U);
      if (i + U < mine) look(b, i + U);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) take(single[j], pieces * 4 + tid + SMP_THREADS * j);
  const unsigned long long own = cand_key(m, last);
  {
    unsigned long long g = own;
#define FIRST_ROW_MAX(CTRL)                                                                                       \
  {                                                                                                               \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(g >> 32), CTRL, 0xf, 0xf, false); \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)g, CTRL, 0xf, 0xf, false);         \
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;                                             \
    g = o > g ? o : g;                                                                                            \
  }
    FIRST_ROW_MAX(0xB1) FIRST_ROW_MAX(0x4E) FIRST_ROW_MAX(0x141) FIRST_ROW_MAX(0x140)
#undef FIRST_ROW_MAX
    if ((lane & 15) == 0) groups[tid >> 4] = g;
  }
  __syncthreads();
  {
    const unsigned long long g = groups[lane];
#pragma unroll
    for (int i = 0; i < 64 / NW; ++i) {           // the places of some of the groups
      const unsigned long long x = groups[wave * (64 / NW) + i];
      if (__popcll(__ballot(g > x)) == k - 1 && lane == 0) bound = x;      // (several zeros in k-th place: all write the same)
    }
  }
  __syncthreads();
  const unsigned long long t = bound;
  auto finish = [&]() __attribute__((always_inline)) {   // wave 0: the draw, or the part's list
    if constexpr (FINAL) {
      if ((draw() && ...)) smp_draw_wave(top, k, temperature, u, token_out + seq, cand_out ? cand_out + (size_t)seq * k : nullptr);
    } else if (lane < k) {
      Cand c = cand_of(top[lane]);
      if (c.i != SMP_NONE) c.i += c0;
      part[((size_t)seq * gridDim.x + blockIdx.x) * k + lane] = c;
    }
  };
  if (k == 1) {                                          // the bound's thread knows the piece
    if (own != 0ull && own == t) {
      if (last < pieces * 4) {
        const Logits4 x = *reinterpret_cast<const Logits4*>(row + last - 3);
        last -= x.v[0] == m ? 3 : x.v[1] == m ? 2 : x.v[2] == m ? 1 : 0;
      }
      top[0] = cand_key(m, last);
    }
    __syncthreads();
    if (wave == 0) finish();
    return;
  }
  if (own != 0ull && own >= t) {
    const float least = cand_of(t).v;
    auto keep = [&](float v, int idx) __attribute__((always_inline)) {
      if (!(v >= least)) return;
      const unsigned long long key = cand_key(v, idx);
      if (key >= t) {
        const int at = atomicAdd(&found, 1);
        if (at < SMP_LIST) list[at] = key;
      }
    };
    for (int i = 0; i < mine; i += 8) {
      Logits4 a[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) a[j] = *reinterpret_cast<const Logits4*>(row + 4 * (tid + SMP_THREADS * min(i + j, mine - 1)));
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (i + j < mine)
#pragma unroll
          for (int e = 0; e < 4; ++e) keep(a[j].v[e], 4 * (tid + SMP_THREADS * (i + j)) + e);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) keep(single[j], pieces * 4 + tid + SMP_THREADS * j);
  }
  __syncthreads();
  if (found <= SMP_LIST) {
    rank_keys(list, found, k, top);
  } else {
    unsigned long long prev = ~0ull;
    for (int r = 0; r < k; ++r) {
      unsigned long long best = 0ull;
      for (int i = tid; i < len; i += SMP_THREADS) {
        const unsigned long long x = cand_key(row[i], i);
        if (x < prev && x > best) best = x;
      }
      const uint32_t hi = wave_max_u32((uint32_t)(best >> 32));
      const uint32_t lo = wave_max_u32((uint32_t)(best >> 32) == hi ? (uint32_t)best : 0u);
      if (lane == 0) groups[wave] = ((unsigned long long)hi << 32) | lo;
      __syncthreads();
      prev = groups[0];
      for (int w = 1; w < NW; ++w) prev = groups[w] > prev ? groups[w] : prev;
      if (tid == 0) top[r] = prev;
      __syncthreads();
    }
  }
  __syncthreads();
  if (wave == 0) finish();
}

// Stage 2: grid (rows).  n candidates of the row, 1024 at a time beside the first k of those before them.
template <typename... Draw>
__global__ void __launch_bounds__(SMP_THREADS) k_topk_draw(const Cand* __restrict__ part, int n, int k, float temperature,
                                                          const float* __restrict__ uniforms, int* __restrict__ token_out,
                                                          int* __restrict__ cand_out, Draw... draw) {
  __shared__ __align__(16) unsigned long long list[SMP_THREADS + SMP_KMAX], top[SMP_KMAX];
  const int tid = threadIdx.x, seq = blockIdx.x;
  const Cand* c = part + (size_t)seq * n;
  const float u = uniforms[seq];
  if (tid < SMP_KMAX) top[tid] = 0ull;
  for (int base = 0; base < n; base += SMP_THREADS) {
    const int now = min(SMP_THREADS, n - base);
    __syncthreads();
    if (tid < now) {
      const Cand x = c[base + tid];
      list[tid] = cand_key(x.v, x.i);
    }
    const unsigned long long before = tid < k ? top[tid] : 0ull;
    if (tid < k) list[now + tid] = before;
    __syncthreads();
    if (tid < k) top[tid] = 0ull;
    __syncthreads();
    rank_keys(list, now + (base > 0 ? k : 0), k, top);
  }
  __syncthreads();
  if (tid < 64 && (draw() && ...)) smp_draw_wave(top, k, temperature, u, token_out + seq, cand_out ? cand_out + (size_t)seq * k : nullptr);
}

}  // namespace first
