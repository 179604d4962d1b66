// A whole decode step of a small full-precision model as one launch per sequence.
//
// What bounds such a step is latency: five dependent mat-vecs and an attention per layer over weights that a few dozen
// compute units read in a microsecond, so that a launch per op spends its time starting and draining (two layers of 256 x 688, 30
// tokens: 61 us a step in 12 launches, 27 here: 9 exchanges of 3 us, half of it the store, the poll and its way back, the other half the
// instructions in between, at some 5 cycles each for a wave that is alone).  So what counts in here is the number of exchanges and of instructions in a
// row: accesses say which memory they mean (through generic pointers every wait for LDS waited for the loads in flight as well), the gains, page ids
// and next layer's pointers are there before they are asked for, the sums of four units meet in the same few lane exchanges.  (36.5 us
// without all that; a second and third poll under way at a time: 9 us a step slower over four layers, everybody reads the same few lines.)
// The workgroups stay and hand vectors to each other through memory:
// every element travels as a 64-bit word {value, epoch}, stored at once; whoever needs the vector loads it until all its words carry the
// epoch it waits for.  Within a launch every vector has the next epoch, and the last one of a launch is kept in device memory for the
// launch that follows.  No vector ever has epoch 0: a launch whose epochs would not all lie below 2^32 begins again at 1 (after hours of
// steps; every word then carries an epoch of the launches just before, far from 1, or a layer's has not been written in that whole cycle).
//
// A word is never overwritten before everyone has read it: whoever writes it again has seen a complete vector since to which EVERY workgroup contributed
// after reading it (each owns at least one row of each mat-vec, see small_step_wgs).  Where attention's output goes round, the residual h is written twice a
// layer, behind the projections and attention's output and behind the MLP's activation.  Where the heads' shares of the output projection go round (BY_HEAD), h is
// written once a layer, behind the MLP's activation, which every workgroup stores after it has read h and the shares; the shares are written again by workgroups that have seen the
// next layer's projections of their head, stored by workgroups that had seen the whole h of the layer before.
//
// Weights of a wave's first rows are requested before it waits for the vector they are multiplied with; the keys and values of a wave's
// first tile before it waits for the queries.  The waits are bounded as in the persistent kernel (sk_poll_give_up).
#pragma once
#include "step_kernel.h"

namespace first {

constexpr int SS_THREADS = 256, SS_WAVES = SS_THREADS / 64;
constexpr int SS_CH = 4;                 // 1 KB pieces of a row (256 elements) requested ahead
// Where the line lies, us a step of two layers, launch per op / this kernel as it was when the line was drawn: widths 256 / 688 at 30 tokens 61.0 / 37.6,
// 1000 92.8 / 64.4, 2000 107.8 / 92.4, 4000 142 / 156 (one workgroup a head walks the keys); 512 / 1536 at 30 tokens 89.9 / 67.5, 2000 141 / 126;
// 1024 / 2816 120.5 / 120.5 and 1024 / 4096 183 / 248 (64 compute units read 4.2 TB/s, the others' share is missed).  Since then, four layers, before / after:
// 256 / 688 at 30 tokens 64.7 / 46.5, 1000 127.5 / 102.7, 2000 181 / 150; 512 / 1376, 8 heads, at 30 tokens 104.5 / 87; 4 heads of 128 at 100 115.5 / 96.
constexpr int SS_MAX_D = 512, SS_MAX_F = 2048, SS_MAX_SEQ = 2048, SS_MAX_V = 16384;
// Four waves, 128 registers and at most 23 KB of LDS: one such workgroup fits on a compute unit beside one of the persistent kernel (eight waves
// of at most 192 registers, up to 133 KB), so 256 of them, four steps, find room beside a persistent kernel that holds every compute
// unit.  Kernels whose workgroups wait for each other then never wait for each other's places; step_order.h sees to the four, and to persistent
// kernels that take more LDS; the build refuses more registers of either kernel.  The compiler keeps to 128 registers by spilling some
// twenty (84 to 104 bytes of scratch a lane; its own loads, none of them in flight); 512 threads and 254 registers would leave no room.
constexpr size_t SS_MAX_LDS = 23 * 1024;
typedef unsigned long long ss_word;
// Where each head's share of the output projection goes round instead of its output (BY_HEAD), and whoever reads the residual adds the shares up: up to four
// words an element, at most an element a thread.  Four layers of 256 / 688 at 30 tokens 58.7 us a step without, 55.0 with it; 512 / 1376 with 8 heads 91.1 / 96.2
// and with 4 heads of 128 102.2 / 108.7 (sixteen words a thread).
constexpr int SS_HEADS = 4;
__host__ __device__ constexpr bool ss_by_head(int Hq, int D) { return Hq <= SS_HEADS && D <= SS_THREADS; }

struct SmallStep {
  DecParams d;                           // geometry, state of sequence d.b, embedding, head (no layer)
  const LayerDev* layers;                // (fp32 matrices and pools behind the pointers)
  const int *kept, *n_kept;
  int L;
  ss_word *xh, *xqkv, *xattn, *xz, *xcand;
  unsigned* epoch;                       // the last epoch of the launches before
  int* err;
};
__host__ __device__ constexpr size_t ss_lds_floats(int D, int nq, int F, int hd) {
  const int k = D > nq ? (D > F ? D : F) : (nq > F ? nq : F);
  return (size_t)D + 2 * k + 2 * SS_WAVES + 4 * hd + SS_WAVES * (hd + 2) + 2 * SS_WAVES + 4;
}

__device__ __forceinline__ void ss_put(ss_word* p, float v, unsigned epoch) {
  __hip_atomic_store(as_global(p), ((ss_word)epoch << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The same value, of which the compiler does not know it: what is computed from it stays in the loop over the layers (hoisted out of it, the
// offsets of all phases took more registers than there are).
__device__ __forceinline__ int ss_fresh(int v) { asm volatile("" : "+v"(v)); return v; }
// The wave's words at(0) .. at(W - 1), once all of them carry the epoch, in v.  False: gave up.
template <int W, typename At>
__device__ __forceinline__ bool ss_wait(At at, unsigned epoch, int* err, float (&v)[W]) {
  unsigned spins = 0;
  for (;;) {
    ss_word a[W];
    bool there = true;
#pragma unroll
    for (int u = 0; u < W; ++u) a[u] = __hip_atomic_load(as_global(at(u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int e = __hip_atomic_load(as_global(err), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int u = 0; u < W; ++u) there = there && (unsigned)(a[u] >> 32) == epoch;
    if (__all(there)) {
#pragma unroll
      for (int u = 0; u < W; ++u) v[u] = __uint_as_float((uint32_t)a[u]);
      return true;
    }
    if (sk_poll_give_up(spins, uni(e), err)) return false;
  }
}
// use(i, value) for this thread's words src(0) .. src(n - 1), once they carry the epoch; W of them at a time.  False: gave up.
template <int W, typename S, typename F>
__device__ __forceinline__ bool ss_get_w(S src, int n, unsigned epoch, int* err, F use) {
  for (int i0 = 0; i0 < n; i0 += W * SS_THREADS) {
    const int i = i0 + ss_fresh(threadIdx.x);
    float v[W];
    if (!ss_wait<W>([&](int u) __attribute__((always_inline)) { return src(min(i + u * SS_THREADS, n - 1)); }, epoch, err, v)) return false;
#pragma unroll
    for (int u = 0; u < W; ++u)
      if (i + u * SS_THREADS < n) use(i + u * SS_THREADS, v[u]);
  }
  return true;
}
template <typename F>
__device__ __forceinline__ bool ss_get(const ss_word* src, int n, unsigned epoch, int* err, F use) {
  auto at = [=](int i) __attribute__((always_inline)) { return src + i; };
  return n <= SS_THREADS ? ss_get_w<1>(at, n, epoch, err, use) : ss_get_w<4>(at, n, epoch, err, use);
}
__device__ __forceinline__ float all_lanes_sum(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum_lane63(v)), 63));
}

// a of the lower and b of the upper half of the wave (row pairs: of the even and the odd row of sixteen lanes), each added over both halves.
__device__ __forceinline__ float ss_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float ss_row_pairs(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float ss_row16(float v) { v = dpp_add<0xB1, 0xf>(v); v = dpp_add<0x4E, 0xf>(v); v = dpp_add<0x141, 0xf>(v); return dpp_add<0x140, 0xf>(v); }

// NR dot products per unit, units dealt to the waves of the grid workgroup first: epi(unit, sums) in a lane of the unit's own.  As many of a wave's units as
// SS_CH pieces of a row hold are requested together (four rows of 256 elements, two of 512), the first ones before the vector is waited
// for: with one row at a time every further one cost a memory round trip (41.3 us a step against 36.5).  stage() brings the vector into xs
// (and ends with a barrier); false: a wait gave up.
template <int NR, typename RowPtr, typename Stage, typename Epi>
__device__ __forceinline__ bool ss_rows(int units, int K, int xs, RowPtr row, Stage stage, Epi epi) {
  extern __shared__ __align__(16) float smem_f[];
  static_assert(SS_CH == 4, "one, two or four units in the pieces below");
  const int lane = ss_fresh(threadIdx.x & 63), step = gridDim.x * SS_WAVES;
  const int np = (K + 255) / 256, together = np == 1 ? 4 : np == 2 ? 2 : 1;      // pieces of a row; units at a time
  int u = uni((int)((threadIdx.x >> 6) * gridDim.x + blockIdx.x));
  f32x4_t w[SS_CH][NR];
  auto k_of = [&](int c) __attribute__((always_inline)) { return ((together == 4 ? 0 : together == 2 ? c & 1 : c) * 64 + lane) * 4; };
  auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < SS_CH; ++c) {
      const int unit = min(u + (together == 4 ? c : together == 2 ? c >> 1 : 0) * step, units - 1);
#pragma unroll
      for (int j = 0; j < NR; ++j) w[c][j] = *as_global(reinterpret_cast<const f32x4_t*>(row(unit, j) + min(k_of(c), K - 4)));
    }
  };
  fetch();
  if (!stage()) return false;
  for (; u < units; u += together * step) {
    float s[SS_CH][NR];
    auto dot = [&](const f32x4_t& a, int k, float t) __attribute__((always_inline)) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(smem_f + xs + k);
      t = fmaf(a.x, x.x, t); t = fmaf(a.y, x.y, t); t = fmaf(a.z, x.z, t);
      return fmaf(a.w, x.w, t);
    };
#pragma unroll
    for (int c = 0; c < SS_CH; ++c)
#pragma unroll
      for (int j = 0; j < NR; ++j) s[c][j] = k_of(c) < K ? dot(w[c][j], k_of(c), 0.f) : 0.f;
    for (int k = (SS_CH * 64 + lane) * 4; k < K; k += 256)
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const f32x4_t more = *as_global(reinterpret_cast<const f32x4_t*>(row(u, j) + k));
        s[0][j] = dot(more, k, s[0][j]);
      }
    const int u0 = u;
    if (u + together * step < units) { u += together * step; fetch(); u = u0; }
    // The four sums of a row of units at once, sixteen lanes for each in the end: 3 exchanges and 4 steps within the lanes instead of 4 times 6, and one
    // epilogue for all of them.
    float t[NR];
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      if (together == 2) { s[0][j] += s[1][j]; s[1][j] = s[2][j] + s[3][j]; s[2][j] = s[0][j]; s[3][j] = s[1][j]; }
      if (together == 1) s[0][j] = s[1][j] = s[2][j] = s[3][j] = (s[0][j] + s[1][j]) + (s[2][j] + s[3][j]);
      t[j] = ss_row16(ss_row_pairs(ss_halves(s[0][j], s[1][j]), ss_halves(s[2][j], s[3][j])));
    }
    const int mine = (lane >> 5) | ((lane >> 3) & 2), unit = u0 + mine * step;       // (the rows of lanes have units 0, 2, 1, 3)
    if ((lane & 15) == 0 && mine < together && unit < units) epi(unit, t);
  }
  return true;
}

__device__ __forceinline__ SmallStep ss_params() { return sk_const<SmallStep>(sk_args()); }

// BY_HEAD: see SS_HEADS.  A group of workgroups walks the keys of each head, all of them alike, and each multiplies what comes out with its rows of the output
// projection's columns of that head: one exchange less than if the heads' outputs went round first.
template <int HD, bool BY_HEAD>
__global__ void __launch_bounds__(SS_THREADS, 4) k_small_step(SmallStep) {
  extern __shared__ __align__(16) float smem_f[];
  constexpr int HALF = HD / 2, KT = 2048 / HD;        // keys of a tile: a lane has 32 dims of one
  constexpr int VL = HD / 4, SUB = 64 / VL;          // lanes that a value row takes, value rows of a request
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, wg = blockIdx.x;
  // (the kernel's arguments are read where they are needed: kept through all phases they are more than there are scalar registers)
  const int D = uni(ss_params().d.D), nq = uni(ss_params().d.Hq * HD), kmax = max(D, max(nq, uni(ss_params().d.F)));
  // LDS: the residual, the vector that is multiplied (two in turn: a wave may still read the one before), ...
  const int x_first = D, red = D + 2 * kmax;
  float* hbuf = smem_f;
  float* qs = smem_f + red + 2 * SS_WAVES;
  float *kn = qs + HD, *vn = kn + HD;
  float2* cs = reinterpret_cast<float2*>(vn + HD);
  float* parts = vn + 2 * HD;                          // [wave][HD dims, max, sum]
  Best* wbest = reinterpret_cast<Best*>(parts + SS_WAVES * (HD + 2));
  int* bad = reinterpret_cast<int*>(wbest + SS_WAVES);
  int pos, n_kept, b;
  unsigned ep;
  {
    const SmallStep P = ss_params();
    const DecParams& p = P.d;
    b = uni(p.b);
    if (__hip_atomic_load(as_global(P.err), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1) return;
    pos = uni(*as_global(p.len + b)); n_kept = uni(*as_global(P.n_kept + b));
    const int tok = min(max(uni(*as_global(p.tokens + b)), 0), p.V - 1);
    ep = (unsigned)uni((int)*as_global(P.epoch));
    for (int i = tid; i < D; i += SS_THREADS) hbuf[i] = ldg(reinterpret_cast<const float*>(p.embed) + (size_t)tok * D + i);
  }
  if (ep > ~0u - (5u * n_kept + 1u)) ep = 0u;        // (five epochs a layer, one for the candidates)
  // a query head each for workgroups 0 .. Hq - 1, or for as many times Hq as there are
  const int Hq = nq / HD, group = BY_HEAD ? (int)gridDim.x / Hq : 1, member = BY_HEAD ? wg / Hq : 0, head = BY_HEAD ? wg - member * Hq : wg;
  const bool attends = BY_HEAD ? member < group : wg < Hq;
  if (tid == 0) *bad = 0;
  // page and row of a lane's key of tile t.  (Keys that are not in the cache - this step's, and those behind it - are clamped to one that is, and replaced.)
  // A tile ahead of the keys; a wave's first one stands at the same place of all layers' pools.
  auto page_of = [&](const SmallStep& P, int t, int& page, int& row) __attribute__((always_inline)) {
    const int key = min(t * KT + ss_fresh(lane) % KT, max(pos - 1, 0)), at = key / P.d.P;
    row = key - at * P.d.P;
    page = *as_global(P.d.page_table + (size_t)b * P.d.max_pages + at);
  };
  int first_off = 0;
  if (attends) {
    const SmallStep P = ss_params();
    int page, row;
    page_of(P, min(wave, pos / KT), page, row);
    first_off = page * (int)P.d.page_elems + row * HD;
  }
  __syncthreads();

  int turn = 0;
  int xs = x_first;
  float rms = 0.f;
  // xs = x * gain of the residual of this epoch (0, nobody's: the embedding, which is in hbuf), and what 1/rms multiplies the results with
  // (heads: it is hbuf plus the heads' shares in xo)
  auto stage_norm = [&](const SmallStep& P, const float* gain, unsigned epoch, bool heads) __attribute__((always_inline)) {
    float ss = 0.f;
    const int t0 = ss_fresh(tid), i1 = t0 + SS_THREADS;
    const float g0 = ldg(gain + min(t0, D - 1)), g1 = D > SS_THREADS ? ldg(gain + min(i1, D - 1)) : 0.f;     // (requested before the residual is waited for)
    auto take = [&](int i, float v) __attribute__((always_inline)) { hbuf[i] = v; smem_f[xs + i] = v * (i < SS_THREADS ? g0 : g1); ss = fmaf(v, v, ss); };
    if (epoch == 0) {
      for (int i = t0; i < D; i += SS_THREADS) take(i, hbuf[i]);
    } else if (heads) {
      float v[SS_HEADS];
      const bool ok = ss_wait<SS_HEADS>([&](int u) __attribute__((always_inline)) { return P.xattn + min(u, Hq - 1) * D + min(t0, D - 1); }, epoch, P.err, v);
      float s = v[0];
#pragma unroll
      for (int u = 1; u < SS_HEADS; ++u) s += u < Hq ? v[u] : 0.f;
      if (t0 < D) take(t0, hbuf[t0] + s);
      if (!ok) *bad = 1;
    } else if (!ss_get(P.xh, D, epoch, P.err, take)) {
      *bad = 1;
    }
    ss = all_lanes_sum(ss);
    if (lane == 0) smem_f[red + turn * SS_WAVES + wave] = ss;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < SS_WAVES; ++w) t += smem_f[red + turn * SS_WAVES + w];
    rms = 1.0f / sqrtf(t / (float)D + P.d.eps);
    return *bad == 0;
  };
  auto stage_plain = [&](const SmallStep& P, const ss_word* src, int n, unsigned epoch) __attribute__((always_inline)) {
    if (!ss_get(src, n, epoch, P.err, [&](int i, float v) __attribute__((always_inline)) { smem_f[xs + i] = v; })) *bad = 1;
    __syncthreads();
    return *bad == 0;
  };
  auto next = [&]() __attribute__((always_inline)) { turn ^= 1; xs = x_first + turn * kmax; };

  unsigned ep_h = 0;                                 // epoch of the residual that the next norm reads
  auto table_of = [&](int kl) __attribute__((always_inline)) {
    const SmallStep P = ss_params();
    return sk_uniform(reinterpret_cast<unsigned long long>(P.layers + uni(*as_global(P.kept + (size_t)b * P.L + kl))));
  };
  unsigned long long at_next = n_kept > 0 ? table_of(0) : 0;
  for (int kl = 0; kl < n_kept; ++kl) {
    const unsigned long long at = at_next;             // of the layers' table
    const unsigned e_qkv = ep + 1, e_attn = ep + 2, e_o = ep + 3, e_z = ep + 4, e_d = ep + 5;
    ep += 5;
    {
      const SmallStep P = ss_params();
      const LayerDev l = sk_const<LayerDev>(at);
      const float *wq = reinterpret_cast<const float*>(l.wq), *wk = reinterpret_cast<const float*>(l.wk), *wv = reinterpret_cast<const float*>(l.wv);
      const int nkv = P.d.Hkv * HD;
      if (!ss_rows<1>(nq + 2 * nkv, D, xs,
                      [&](int r, int) __attribute__((always_inline)) { return r < nq ? wq + (size_t)r * D : r < nq + nkv ? wk + (size_t)(r - nq) * D : wv + (size_t)(r - nq - nkv) * D; },
                      [&]() __attribute__((always_inline)) { return stage_norm(P, l.g_attn, ep_h, false); }, [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xqkv + r, s[0] * rms, e_qkv); }))
        return;
    }
    next();
    if (attends) {
      const SmallStep P = ss_params();
      const DecParams& p = P.d;
      const LayerDev l = sk_const<LayerDev>(at);
      const float* wo = reinterpret_cast<const float*>(l.wo);
      float* pool = reinterpret_cast<float*>(l.kv);
      const int nkv = p.Hkv * HD, g = head / p.G;
      const size_t head_off = (size_t)g * p.P * HD, v_off = (size_t)p.Hkv * p.P * HD;
      const SK_GLOBAL int* pt = as_global(p.page_table + (size_t)b * p.max_pages);
      const int tiles = pos / KT + 1;
      // (a lane's key of a tile, its share of that key's dims, its value rows and dims are made where they are used: kept, they cost the walk its registers)
      f32x4_t kf[8];                                 // dims 32 part .. + 32 of this lane's key
      f32x4_t vf[8];                                 // dims 4 vd .. + 4 of keys SUB i + sub
      int off = first_off, page = 0, row = 0;        // where this lane's key of the tile is; page and row of the one that follows
      // (a pool has fewer than 2^31 elements)
      auto fetch_k = [&]() __attribute__((always_inline)) {
        const float* kp = pool + head_off + off + 32 * (ss_fresh(lane) / KT);
#pragma unroll
        for (int c = 0; c < 8; ++c) kf[c] = *as_global(reinterpret_cast<const f32x4_t*>(kp + 4 * c));
      };
      auto fetch_v = [&]() __attribute__((always_inline)) {
        const int ln = ss_fresh(lane), sub = ln / VL;
        const float* values = pool + head_off + v_off + 4 * (ln % VL);
#pragma unroll
        for (int i = 0; i < 8; ++i) vf[i] = *as_global(reinterpret_cast<const f32x4_t*>(values + __builtin_amdgcn_ds_bpermute(4 * sub + 4 * SUB * i, off)));
      };
      const int sub = ss_fresh(lane) / VL, vd = ss_fresh(lane) % VL;
      // rows of the output projection of this workgroup: SUB a wave at a time, NO times requested ahead
      constexpr int NO = HD / 64;
      const int o0 = BY_HEAD ? D * member / group : 0, o1 = BY_HEAD ? D * (member + 1) / group : 0;
      f32x4_t wf[NO];
      auto o_row = [&](int i) __attribute__((always_inline)) { return o0 + (i * SS_WAVES + wave) * SUB + sub; };
      auto fetch_o = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NO; ++i) wf[i] = *as_global(reinterpret_cast<const f32x4_t*>(wo + (size_t)min(o_row(i0 + i), o1 - 1) * nq + head * HD + 4 * vd));
      };
      fetch_k();                                     // (a wave without a tile loads one all the same: no branch around 64 registers)
      fetch_v();
      if (wave + SS_WAVES < tiles) page_of(P, wave + SS_WAVES, page, row);
      if (kl == 0 && tid < HALF) {                   // (behind the first projections: nobody waits for it there)
        const double a = (double)pos * *as_global(p.theta + tid);
        cs[tid] = make_float2((float)cos(a), (float)sin(a));
      }
      // q, k, v of the head: qs, kn, vn raw; rotated in place behind the barrier
      const int xq = head * HD, xk = nq + g * HD;
      const bool ok = ss_get_w<(3 * HD + SS_THREADS - 1) / SS_THREADS>([=](int i) __attribute__((always_inline)) { return P.xqkv + (i < HD ? xq + i : i < 2 * HD ? xk + (i - HD) : xk + (nkv + i - 2 * HD)); },
                                                                       3 * HD, e_qkv, P.err, [&](int i, float v) __attribute__((always_inline)) { qs[i] = v; });
      if (!ok) *bad = 1;
      __syncthreads();
      if (*bad) return;
      if (tid < HD) {
        const int d = tid % HALF;
        float* x = tid < HALF ? qs : kn;
        const float x1 = x[d], x2 = x[d + HALF];
        const float2 c = cs[d];
        const float sc = tid < HALF ? p.qscale : 1.f;
        x[d] = (x1 * c.x - x2 * c.y) * sc;
        x[d + HALF] = (x2 * c.x + x1 * c.y) * sc;
      }
      __syncthreads();
      if (member == 0 && head == g * p.G && tid < HD) {             // one head of the group appends the new position
        float* dst = pool + (size_t)pt[pos / p.P] * p.page_elems + head_off + (size_t)(pos % p.P) * HD + tid;
        *as_global(dst) = kn[tid];
        *as_global(dst + v_off) = vn[tid];
      }
      float m = -INFINITY, sum = 0.f;
      f32x4_t o = {0.f, 0.f, 0.f, 0.f};
      for (int t = wave; t < tiles;) {
        const int ln = ss_fresh(lane), klane = ln % KT, part = ln / KT, sub = ln / VL, vd = ln % VL;
        const int k0 = t * KT, key = k0 + klane, d0 = 32 * part;
        if (t == tiles - 1) {                        // the new position, and what is behind it (weight 0)
          if (key >= pos) {
#pragma unroll
            for (int c = 0; c < 8; ++c) kf[c] = *reinterpret_cast<const f32x4_t*>(kn + d0 + 4 * c);
          }
          const f32x4_t v_new = *reinterpret_cast<const f32x4_t*>(vn + 4 * vd);
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (k0 + SUB * i + sub >= pos) vf[i] = v_new;
        }
        float sc = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const f32x4_t q4 = *reinterpret_cast<const f32x4_t*>(qs + d0 + 4 * c);
#pragma unroll
          for (int e = 0; e < 4; ++e) sc = fmaf(q4[e], kf[c][e], sc);
        }
        if (HD == 128) sc = ss_row_pairs(sc, sc);
        sc = ss_halves(sc, sc);
        const bool more = t + SS_WAVES < tiles;
        if (more) {                                  // (the keys have been used: the next tile's, while the weights are made and the values added)
          off = page * (int)p.page_elems + row * HD;
          fetch_k();
          if (t + 2 * SS_WAVES < tiles) page_of(P, t + 2 * SS_WAVES, page, row);
        }
        if (key > pos) sc = -INFINITY;
        const float mn = fmaxf(m, wave_max(sc)), corr = expf(m - mn), pj = key <= pos ? expf(sc - mn) : 0.f;
        sum = sum * corr + all_lanes_sum(part == 0 ? pj : 0.f);
        m = mn;
        o *= corr;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float w = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * sub + 4 * SUB * i, __float_as_int(pj)));
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = fmaf(w, vf[i][e], o[e]);
        }
        t += SS_WAVES;
        if (!more) break;
        fetch_v();
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (SUB == 4) o[e] = ss_row_pairs(o[e], o[e]);
        o[e] = ss_halves(o[e], o[e]);
        if (sub == 0) parts[wave * (HD + 2) + 4 * vd + e] = o[e];
      }
      if (lane == 0) { parts[wave * (HD + 2) + HD] = m; parts[wave * (HD + 2) + HD + 1] = sum; }
      if (BY_HEAD) fetch_o(0);
      __syncthreads();
      if (tid < HD) {
        const int live = min(tiles, SS_WAVES);
        float M = -INFINITY, den = 0.f, num = 0.f;
        for (int w = 0; w < live; ++w) M = fmaxf(M, parts[w * (HD + 2) + HD]);
        for (int w = 0; w < live; ++w) {
          const float c = expf(parts[w * (HD + 2) + HD] - M);
          den = fmaf(parts[w * (HD + 2) + HD + 1], c, den);
          num = fmaf(parts[w * (HD + 2) + tid], c, num);
        }
        if (BY_HEAD) qs[tid] = num / den;
        else ss_put(P.xattn + head * HD + tid, num / den, e_attn);
      }
      if (BY_HEAD) {
        __syncthreads();
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(qs + 4 * vd);
        for (int i0 = 0; o0 + i0 * SS_WAVES * SUB < o1; i0 += NO) {
          if (i0 > 0) fetch_o(i0);
#pragma unroll
          for (int i = 0; i < NO; ++i) {
            float s = wf[i].x * x.x;
            s = fmaf(wf[i].y, x.y, s); s = fmaf(wf[i].z, x.z, s); s = fmaf(wf[i].w, x.w, s);
            s = dpp_add<0xB1, 0xf>(s); s = dpp_add<0x4E, 0xf>(s); s = dpp_add<0x141, 0xf>(s); s = dpp_add<0x140, 0xf>(s);
            if (VL == 32) s += __shfl_xor(s, 16, 64);
            if (vd == 0 && o_row(i0 + i) < o1) ss_put(P.xattn + head * D + o_row(i0 + i), s, e_o);
          }
        }
      }
    }
    if (!BY_HEAD) {
      const SmallStep P = ss_params();
      const float* wo = reinterpret_cast<const float*>(sk_const<LayerDev>(at).wo);
      if (!ss_rows<1>(D, nq, xs, [&](int r, int) __attribute__((always_inline)) { return wo + (size_t)r * nq; }, [&]() __attribute__((always_inline)) { return stage_plain(P, P.xattn, nq, e_attn); },
                      [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xh + r, hbuf[r] + s[0], e_o); }))
        return;
      next();
    }
    unsigned seen;
    {
      const SmallStep P = ss_params();
      const LayerDev l = sk_const<LayerDev>(at);
      const int following = *as_global(P.kept + (size_t)b * P.L + min(kl + 1, n_kept - 1));
      const float *wgt = reinterpret_cast<const float*>(l.wg), *wup = reinterpret_cast<const float*>(l.wu);
      if (!ss_rows<2>(P.d.F, D, xs, [&](int r, int j) __attribute__((always_inline)) { return (j ? wup : wgt) + (size_t)r * D; }, [&]() __attribute__((always_inline)) { return stage_norm(P, l.g_mlp, e_o, BY_HEAD); },
                      [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xz + r, siluf(s[0] * rms) * (s[1] * rms), e_z); }))
        return;
      next();
      // where the next layer's pointers are, and those into the scalar cache: a first look at them costs a memory round trip
      at_next = sk_uniform(reinterpret_cast<unsigned long long>(P.layers + uni(following)));
      seen = sk_const<unsigned>(at_next) | sk_const<unsigned>(at_next + sizeof(LayerDev) - 4);
    }
    {
      const SmallStep P = ss_params();
      const float* wd = reinterpret_cast<const float*>(sk_const<LayerDev>(at).wd);
      const int F = P.d.F;
      if (!ss_rows<1>(D, F, xs, [&](int r, int) __attribute__((always_inline)) { return wd + (size_t)r * F; }, [&]() __attribute__((always_inline)) { return stage_plain(P, P.xz, F, e_z); },
                      [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xh + r, hbuf[r] + s[0], e_d); }))
        return;
      next();
    }
    asm volatile("" : : "s"(seen));
    ep_h = e_d;
  }

  // logits, and the first of the best
  const SmallStep P = ss_params();
  const DecParams& p = P.d;
  Best best{-INFINITY, 0x7fffffff};
  float* lg = p.logits ? p.logits + (size_t)b * p.V : nullptr;
  const float* wl = reinterpret_cast<const float*>(p.lm_head);
  if (!ss_rows<1>(p.V, D, xs, [&](int r, int) __attribute__((always_inline)) { return wl + (size_t)r * D; }, [&]() __attribute__((always_inline)) { return stage_norm(P, p.g_final, ep_h, false); },
                  [&](int r, const float* s) __attribute__((always_inline)) {
                    const Best c{s[0] * rms, r};
                    if (lg) *as_global(lg + r) = c.v;
                    if (better(c, best)) best = c;
                  }))
    return;
  ++ep;
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const Best c{__shfl_xor(best.v, o, 64), __shfl_xor(best.i, o, 64)};
    if (better(c, best)) best = c;
  }
  if (lane == 0) wbest[wave] = best;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < SS_WAVES; ++w) if (better(wbest[w], best)) best = wbest[w];
    ss_put(P.xcand + 2 * wg, best.v, ep);
    ss_put(P.xcand + 2 * wg + 1, __int_as_float(best.i), ep);
  }
  if (wg != 0) return;
  for (int i = tid; i < D; i += SS_THREADS) *as_global(p.h + (size_t)b * D + i) = hbuf[i];
  const bool ok = ss_get(P.xcand, 2 * (int)gridDim.x, ep, P.err, [&](int i, float v) __attribute__((always_inline)) { smem_f[x_first + (turn ^ 1) * kmax + i] = v; });
  if (!ok) *bad = 1;
  __syncthreads();
  if (*bad || wave != 0) return;
  best = Best{-INFINITY, 0x7fffffff};
  for (int i = lane; i < (int)gridDim.x; i += 64) {
    const Best c{smem_f[x_first + (turn ^ 1) * kmax + 2 * i], __float_as_int(smem_f[x_first + (turn ^ 1) * kmax + 2 * i + 1])};
    if (better(c, best)) best = c;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const Best c{__shfl_xor(best.v, o, 64), __shfl_xor(best.i, o, 64)};
    if (better(c, best)) best = c;
  }
  if (lane == 0) {
    if (p.token_out) p.token_out[b] = best.i;
    if (p.advance_len) p.len[b] = pos + 1;
    *P.epoch = ep;
  }
}

}  // namespace first
