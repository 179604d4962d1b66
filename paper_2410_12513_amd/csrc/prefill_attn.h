// Prompt attention on the matrix cores (bf16 cache, head_dim 64 or 128) and the preparation of its operands, for a group of
// prompts at once.
//
// The prompts of a group follow each other in the rows of every activation matrix.  For attention their keys and values
// also stand in copies in which each prompt starts at a multiple of 128 ("padded rows"), laid out so that what a
// workgroup fetches at a time is contiguous:
//   kc [KV head][padded row][hd]             the keys as the cache stores them
//   vt [KV head][tile of 64][hd][64 keys]    the values transposed; the 16 keys of a group stand in the order in which the
//                                            score accumulators hold them (0-3, 8-11, 4-7, 12-15), so that an A operand of
//                                            the second product is one 16-byte read
#pragma once
#include "prefill_gemm.h"
#include "prefill_kernels.h"

namespace first {

constexpr int PACK_PAD = 128;            // padded rows of a prompt are a multiple of this
constexpr int FA_TILE = 64;              // keys per tile of kc / vt
constexpr int FA_WIDE_FROM = 2048;       // prompts of at least this many tokens: 128 queries a workgroup
constexpr float LOG2E = 1.4426950408889634f;

// x in both halves of the wave -> (value of lane % 32 in the lower half, in the upper half)
__device__ __forceinline__ void both_halves(float x, float& lower, float& upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lower = __uint_as_float(r[0]); upper = __uint_as_float(r[1]);
}

// Rotation, splits and cache writes of one head (blockIdx.y: query heads, then key heads, then value heads) for 32 padded rows
// (blockIdx.x).  Queries leave rotated, scaled by qscale and split; keys and
// values go to their pages and to kc / vt.  One pass over the fp32 projections, where a rotation in place, a split of the
// queries and a gather of the pages were three (36 us a layer at 1024 tokens of the 8B shape, 11 now).
template <int HD>
__global__ void __launch_bounds__(WG) k_rope_split(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
                                                   const float2* __restrict__ cs, PromptPack pk, bf16* __restrict__ pool, size_t page_elems,
                                                   bf16* __restrict__ qh, bf16* __restrict__ ql, bf16* __restrict__ kc, bf16* __restrict__ vt,
                                                   int Hq, int Hkv, int padded, int P, float qscale) {
  constexpr int HALF = HD / 2, QP = HALF / 4;               // groups of four dims per half
  __shared__ uint16_t vs[32][HD + 2];
  const int tid = threadIdx.x, p0 = blockIdx.x * 32, y = blockIdx.y;
  const int j = pack_find(pk.poff, pk.n, p0);
  const int t0 = p0 - (pk.poff[j] - pk.poff[0]), r0 = pk.off[j] - pk.off[0], T = pk.off[j + 1] - pk.off[j];
  const int* pt = pk.pt + (size_t)(pk.b0 + j) * pk.max_pages;
  const size_t v_off = (size_t)Hkv * P * HD;
  if (y < Hq + Hkv) {
    const bool isq = y < Hq;
    const int h = isq ? y : y - Hq, pitch = (isq ? Hq : Hkv) * HD;
    const float* src = isq ? q : k;
#pragma unroll
    for (int u = 0; u < 32 * QP / WG; ++u) {
      const int i = tid + WG * u, row = i / QP, d = (i % QP) * 4, t = t0 + row;
      if (t >= T) continue;
      const float* x = src + (size_t)(r0 + t) * pitch + h * HD + d;
      const float4 a = *reinterpret_cast<const float4*>(x), b = *reinterpret_cast<const float4*>(x + HALF);
      const float2* c = cs + (size_t)t * HALF + d;
      const float2 c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
      float lo[4] = {a.x * c0.x - b.x * c0.y, a.y * c1.x - b.y * c1.y, a.z * c2.x - b.z * c2.y, a.w * c3.x - b.w * c3.y};
      float up[4] = {b.x * c0.x + a.x * c0.y, b.y * c1.x + a.y * c1.y, b.z * c2.x + a.z * c2.y, b.w * c3.x + a.w * c3.y};
      if (isq) {
        uint2 h1, l1, h2, l2;
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] *= qscale; up[e] *= qscale; }
        split_pair(lo[0], lo[1], h1.x, l1.x); split_pair(lo[2], lo[3], h1.y, l1.y);
        split_pair(up[0], up[1], h2.x, l2.x); split_pair(up[2], up[3], h2.y, l2.y);
        const size_t o = (size_t)(r0 + t) * pitch + h * HD + d;
        *reinterpret_cast<uint2*>(qh + o) = h1; *reinterpret_cast<uint2*>(qh + o + HALF) = h2;
        *reinterpret_cast<uint2*>(ql + o) = l1; *reinterpret_cast<uint2*>(ql + o + HALF) = l2;
      } else {
        const uint2 k1 = make_uint2(pk_bf16(lo[0], lo[1]), pk_bf16(lo[2], lo[3])), k2 = make_uint2(pk_bf16(up[0], up[1]), pk_bf16(up[2], up[3]));
        bf16* dst = kc + ((size_t)h * padded + p0 + row) * HD + d;
        *reinterpret_cast<uint2*>(dst) = k1; *reinterpret_cast<uint2*>(dst + HALF) = k2;
        bf16* pg = pool + (size_t)pt[t / P] * page_elems + (size_t)h * P * HD + (size_t)(t % P) * HD + d;
        *reinterpret_cast<uint2*>(pg) = k1; *reinterpret_cast<uint2*>(pg + HALF) = k2;
      }
    }
    return;
  }
  const int g = y - Hq - Hkv;
#pragma unroll
  for (int u = 0; u < 32 * HD / 4 / WG; ++u) {
    const int i = tid + WG * u, row = i / (HD / 4), d = (i % (HD / 4)) * 4, t = t0 + row;
    uint2 w = make_uint2(0u, 0u);                           // keys past the end: zeros, whatever weight the scores give them
    if (t < T) {
      const float4 a = *reinterpret_cast<const float4*>(v + (size_t)(r0 + t) * Hkv * HD + g * HD + d);
      w = make_uint2(pk_bf16(a.x, a.y), pk_bf16(a.z, a.w));
      *reinterpret_cast<uint2*>(pool + (size_t)pt[t / P] * page_elems + v_off + (size_t)g * P * HD + (size_t)(t % P) * HD + d) = w;
    }
    vs[row][d] = (uint16_t)w.x; vs[row][d + 1] = (uint16_t)(w.x >> 16);
    vs[row][d + 2] = (uint16_t)w.y; vs[row][d + 3] = (uint16_t)(w.y >> 16);
  }
  __syncthreads();
  bf16* tile = vt + ((size_t)g * padded + (p0 & ~(FA_TILE - 1))) * HD + (p0 & (FA_TILE - 1));
#pragma unroll
  for (int u = 0; u < 4 * HD / WG; ++u) {                   // 16 bytes: eight keys of one dim
    const int i = tid + WG * u, c = i & 3, d = i >> 2, kb = 16 * (c >> 1) + 4 * (c & 1);
    uint4 w;
    w.x = vs[kb][d] | ((uint32_t)vs[kb + 1][d] << 16); w.y = vs[kb + 2][d] | ((uint32_t)vs[kb + 3][d] << 16);
    w.z = vs[kb + 8][d] | ((uint32_t)vs[kb + 9][d] << 16); w.w = vs[kb + 10][d] | ((uint32_t)vs[kb + 11][d] << 16);
    *reinterpret_cast<uint4*>(tile + (size_t)d * FA_TILE + 8 * c) = w;
  }
}

// Causal GQA attention of a group of prompts.
//
// A workgroup takes QG x 32 queries of one head; four waves, QG groups of queries x KH shares of each 64-key tile.  The tile's
// keys and values go from memory straight into LDS, two tiles in the ring.  Everything is computed transposed, so that a
// lane owns ONE query column:
//   S^T[key][q] = K Q^T     (A = key rows, B = query columns; high and low parts of q)
//   O^T[dim][q] = V^T P^T   (A = rows of the transposed values, B = the probabilities straight from the accumulator
//                            registers of S^T, split hi + lo)
// The maximum of a query is per lane plus one exchange with lane ^ 32, the sum stays per lane until the end, and O^T
// is only rescaled when some query's maximum has grown.  The maximum is kept as it enters the exponent, rounded once after
// its product with log2 e: a weight is 2^(S log2 e - m) with one rounding of that difference, and a rescaling 2^(m - m').  (With
// the product rounded anew for every maximum, weights of different tiles differ by 2^-24 of it: 6e-6 at scores of 100.)  Accumulator layout of the 32x32 MFMA: lane l holds column
// l % 32, register r holds row 8 (r / 4) + 4 (l / 32) + r % 4.
// Bound: matrix cores (64 MFMAs of 32 cycles per 64 keys and 32 queries) with the exponentials and splits of the other
// wave of the SIMD beside them.  KH = 2 doubles the workgroups and halves each wave's walk where the prompts are too short
// to fill the chip; KH = 1 moves half the operand bytes.  Workgroups with the longest walks start first, and workgroups that
// follow each other belong to different KV heads, so that an XCD's L2 sees one head's keys where there are eight of them.
// Measured, 8B heads, kernel trace: 16384 tokens 13.9 -> 3.5 ms a layer (1.2 PFLOP/s of matrix work), 1024 tokens 103 -> 35 us (against
// the earlier kernel: one wave per 32 queries, operands from global memory into registers).
template <int HD, int QG, int KH>
__global__ void __launch_bounds__(WG, 2) k_attn_prompt(const bf16* __restrict__ qh, const bf16* __restrict__ ql, const bf16* __restrict__ kc,
                                                       const bf16* __restrict__ vt, bf16* __restrict__ outh, bf16* __restrict__ outl,
                                                       PromptPack pk, int padded, int Hq, int Hkv) {
  static_assert(QG * KH == WAVES, "four waves");
  constexpr int KS = HD / 16, DT = HD / 32, QB = 32 * QG, KT = FA_TILE / KH, NS = KT / 32;
  constexpr int KB = FA_TILE * HD * 2, STG = 2 * KB;       // bytes of a key tile (= of a value tile), of a stage
  constexpr int NI = KB / 1024 / WAVES;                    // 1 KB loads per wave and operand
  constexpr int KC = HD / 8;                               // 16-byte chunks per key row
  extern __shared__ __align__(16) char fa_smem[];
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)fa_smem;
  const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63, col = lane & 31, gl = lane >> 5;
  const int G = Hq / Hkv, g = blockIdx.x % Hkv, hr = blockIdx.x / Hkv, h = g * G + hr % G;
  const int p0 = (padded / QB - 1 - hr / G) * QB;          // first padded row of this block of queries
  const int j = pack_find(pk.poff, pk.n, p0);
  const int pj = pk.poff[j] - pk.poff[0], r0 = pk.off[j] - pk.off[0], T = pk.off[j + 1] - pk.off[j];
  const int q0 = p0 - pj;
  if (q0 >= T || (KH == 1) != (T >= FA_WIDE_FROM)) return;
  const int qw = q0 + (wave % QG) * 32, kh = wave / QG;    // this wave's queries, its share of a tile
  const bool live = qw < T;
  const int nq = Hq * HD;
  const int qi = qw + col, qc = min(qi, T - 1);

  bf16x8_t Qh[KS], Ql[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const size_t o = (size_t)(r0 + qc) * nq + h * HD + 16 * s + 8 * gl;
    Qh[s] = *reinterpret_cast<const bf16x8_t*>(qh + o);
    Ql[s] = *reinterpret_cast<const bf16x8_t*>(ql + o);
  }
  // what this lane fetches of a tile: key rows of 2 HD bytes, value rows of 128 bytes, chunks permuted by row (bank conflicts)
  auto kslot = [](int row, int c) { return HD == 128 ? c ^ (row & 15) : pg_chunk(row, c); };
  uint32_t vk[NI], vv[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = (wave * NI + i) * 64 + lane;
    vk[i] = (uint32_t)((c / KC) * HD * 2 + kslot(c / KC, c % KC) * 16);
    vv[i] = (uint32_t)((c / 8) * 128 + pg_chunk(c / 8, c % 8) * 16);
  }
  const size_t base = ((size_t)g * padded + pj) * HD;
  auto issue = [&](int st) __attribute__((always_inline)) {
    const i32x4_t rk = pg_rsrc(kc + base + (size_t)st * FA_TILE * HD, KB), rv = pg_rsrc(vt + base + (size_t)st * FA_TILE * HD, KB);
    const uint32_t b = (uint32_t)uni((int)(lds0 + (uint32_t)(st & 1) * STG));
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      pg_load_lds(b + (wave * NI + i) * 1024, vk[i], rk, 0u);
      pg_load_lds(b + KB + (wave * NI + i) * 1024, vv[i], rv, 0u);
    }
  };
  floatx16_t O[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[t][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  const int n_st = (min(q0 + QB, T) + FA_TILE - 1) / FA_TILE;
  const int q_last = min(qw + 31, T - 1);
  issue(0);
  for (int st = 0; st < n_st; ++st) {
    pg_wait<0>();
    lds_barrier();
    if (st + 1 < n_st) issue(st + 1);
    const int k0 = st * FA_TILE + kh * KT;
    if (!live || k0 > q_last) continue;                    // (k0 and qw are multiples of 32: a tile that is not skipped has a key for every query)
    const char* sk = fa_smem + (st & 1) * STG;
    const char* sv = sk + KB;
    floatx16_t S[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) S[u][r] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      bf16x8_t kf[NS];
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int row = kh * KT + 32 * u + col;
        kf[u] = *reinterpret_cast<const bf16x8_t*>(sk + row * HD * 2 + kslot(row, 2 * s + gl) * 16);
      }
#pragma unroll
      for (int u = 0; u < NS; ++u) S[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u], Ql[s], S[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < NS; ++u) S[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u], Qh[s], S[u], 0, 0, 0);
    }
    if (k0 + KT - 1 > qw) {                                // the diagonal
#pragma unroll
      for (int u = 0; u < NS; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + 32 * u + 8 * (r >> 2) + 4 * gl + (r & 3) > qi) S[u][r] = -INFINITY;
    }
    float mt = S[0][0];
#pragma unroll
    for (int u = 0; u < NS; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) mt = fmaxf(mt, S[u][r]);
    float ma, mb;
    both_halves(mt, ma, mb);
    const float mn = fmaxf(m, fmaxf(ma, mb) * LOG2E);      // finite: the tile has a key that this query sees
    if (__any(mn > m)) {
      const float corr = __builtin_amdgcn_exp2f(m - mn);
      l *= corr;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[t][r] *= corr;
      m = mn;
    }
    float ls[4] = {0.f, 0.f, 0.f, 0.f};                    // the tile's sum first: a long prompt's l is thousands of terms
#pragma unroll
    for (int u = 0; u < NS; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) { S[u][r] = __builtin_amdgcn_exp2f(fmaf(S[u][r], LOG2E, -m)); ls[r & 3] += S[u][r]; }
    l += (ls[0] + ls[1]) + (ls[2] + ls[3]);
    // O^T += V^T P^T: k-step s2 uses accumulator registers 8 s2 .. 8 s2 + 7 of P as they are
#pragma unroll
    for (int s2 = 0; s2 < 2 * NS; ++s2) {
      union { uint32_t w[4]; bf16x8_t b; } Ph, Pl;
#pragma unroll
      for (int e = 0; e < 4; ++e) split_pair(S[s2 / 2][8 * (s2 & 1) + 2 * e], S[s2 / 2][8 * (s2 & 1) + 2 * e + 1], Ph.w[e], Pl.w[e]);
      bf16x8_t vf[DT];
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const int row = 32 * t + col;
        vf[t] = *reinterpret_cast<const bf16x8_t*>(sv + row * 128 + pg_chunk(row, (kh * KT) / 8 + 2 * s2 + gl) * 16);
      }
#pragma unroll
      for (int t = 0; t < DT; ++t) O[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t], Pl.b, O[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < DT; ++t) O[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t], Ph.b, O[t], 0, 0, 0);
    }
  }
  float la, lb;
  both_halves(l, la, lb);
  l = la + lb;
  if constexpr (KH == 2) {                                 // the two shares of the keys meet in LDS
    float* ex = reinterpret_cast<float*>(fa_smem) + (size_t)(wave % QG) * (16 * DT + 2) * 64 + lane;
    static_assert((size_t)QG * (16 * DT + 2) * 256 <= (size_t)2 * STG, "partial results fit the ring");
    lds_barrier();
    if (kh == 1) {
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) ex[(t * 16 + r) * 64] = O[t][r];
      ex[16 * DT * 64] = m; ex[(16 * DT + 1) * 64] = l;
    }
    lds_barrier();
    if (kh == 1) return;
    const float m2 = ex[16 * DT * 64], l2 = ex[(16 * DT + 1) * 64], mm = fmaxf(m, m2);
    const float c1 = __builtin_amdgcn_exp2f(m - mm), c2 = __builtin_amdgcn_exp2f(m2 - mm);    // (no tile for the second share: m2 = -inf, c2 = 0)
    l = l * c1 + l2 * c2;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) O[t][r] = O[t][r] * c1 + ex[(t * 16 + r) * 64] * c2;
  }
  if (qi < T) {
    const float inv = 1.0f / l;
    const size_t orow = (size_t)(r0 + qi) * nq + h * HD;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        uint2 hi, lo;
        split_pair(O[t][4 * rr] * inv, O[t][4 * rr + 1] * inv, hi.x, lo.x);
        split_pair(O[t][4 * rr + 2] * inv, O[t][4 * rr + 3] * inv, hi.y, lo.y);
        const size_t o = orow + 32 * t + 8 * rr + 4 * gl;
        *reinterpret_cast<uint2*>(outh + o) = hi;
        *reinterpret_cast<uint2*>(outl + o) = lo;
      }
  }
}

}  // namespace first
