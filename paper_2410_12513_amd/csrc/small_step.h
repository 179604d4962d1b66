// A whole decode step of a small full-precision model as one launch per sequence.
//
// What bounds such a step is latency: five dependent mat-vecs and an attention per layer over weights that a few dozen
// compute units read in a microsecond, so that a launch per op spends its time starting and draining (two layers of 256 x 688, 30
// tokens: 61 us a step in 12 launches, 37.6 here, 36.5 of them in the kernel: 11 exchanges of 3.3 us with the work between them).  The workgroups stay and hand vectors to each other through memory:
// every element travels as a 64-bit word {value, epoch}, stored at once; whoever needs the vector loads it until all its words carry the
// epoch it waits for.  Within a launch every vector has the next epoch, and the last one of a launch is kept in device memory for the
// launch that follows.  No vector ever has epoch 0: a launch whose epochs would not all lie below 2^32 begins again at 1 (after hours of
// steps; every word then carries an epoch of the launches just before, far from 1, or a layer's has not been written in that whole cycle).
//
// A word is never overwritten before everyone has read it: each vector is written again one layer later, by workgroups that have
// seen complete vectors since to which EVERY workgroup contributed after reading this one (each owns at least one row
// of each mat-vec, see small_step_wgs).  The residual h is written twice a layer; the MLP's activation lies between, and attention's
// output before.
//
// Weights of a wave's first rows are requested before it waits for the vector they are multiplied with; the keys and values of a wave's
// first tile before it waits for the queries.  The waits are bounded as in the persistent kernel (sk_poll_give_up).
#pragma once
#include "step_kernel.h"

namespace first {

constexpr int SS_THREADS = 256, SS_WAVES = SS_THREADS / 64;
constexpr int SS_CH = 4;                 // 1 KB pieces of a row (256 elements) requested ahead
// Where the line lies, us a step of two layers, launch per op / this kernel: widths 256 / 688 at 30 tokens 61.0 / 37.6, 1000 92.8 / 64.4, 2000
// 107.8 / 92.4, 4000 142 / 156 (one workgroup a head walks the keys); 512 / 1536 at 30 tokens 89.9 / 67.5, 2000 141 / 126; 1024 / 2816 120.5 / 120.5
// and 1024 / 4096 183 / 248 (64 compute units read 4.2 TB/s, the others' share is missed).
constexpr int SS_MAX_D = 512, SS_MAX_F = 2048, SS_MAX_SEQ = 2048, SS_MAX_V = 16384;
// Four waves, 128 registers and at most 23 KB of LDS: one such workgroup fits on a compute unit beside one of the persistent kernel (eight waves
// of at most 192 registers, up to 133 KB), so 256 of them, four steps, find room beside a persistent kernel that holds every compute
// unit.  Kernels whose workgroups wait for each other then never wait for each other's places; step_order.h sees to the four, and to persistent
// kernels that take more LDS; the build refuses more registers of either kernel.  The compiler keeps to 128 registers by spilling (236 bytes of scratch
// a lane at 64 dims a head, 228 at 128; its own loads, none of them in flight); 512 threads and 254 registers spill nothing and took 33 us
// a step instead of 36.5, but left no room.
constexpr size_t SS_MAX_LDS = 23 * 1024;
typedef unsigned long long ss_word;

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
  __hip_atomic_store(p, ((ss_word)epoch << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// use(i, value) for this thread's words src(0) .. src(n - 1), once they carry the epoch; W of them in flight.  False: gave up.
template <int W, typename S, typename F>
__device__ __forceinline__ bool ss_get_w(S src, int n, unsigned epoch, int* err, F use) {
  for (int i = threadIdx.x; i < n; i += W * SS_THREADS) {
    unsigned spins = 0;
    ss_word a[W];
    for (;;) {
      bool there = true;
#pragma unroll
      for (int u = 0; u < W; ++u) a[u] = __hip_atomic_load(src(min(i + u * SS_THREADS, n - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int e = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < W; ++u) there = there && (unsigned)(a[u] >> 32) == epoch;
      if (there) break;
      if (sk_poll_give_up(spins, e, err)) return false;
    }
#pragma unroll
    for (int u = 0; u < W; ++u)
      if (i + u * SS_THREADS < n) use(i + u * SS_THREADS, __uint_as_float((uint32_t)a[u]));
  }
  return true;
}
template <typename F>
__device__ __forceinline__ bool ss_get(const ss_word* src, int n, unsigned epoch, int* err, F use) {
  auto at = [=](int i) __attribute__((always_inline)) { return src + i; };
  return n <= SS_THREADS ? ss_get_w<1>(at, n, epoch, err, use) : ss_get_w<4>(at, n, epoch, err, use);
}
// The same value, of which the compiler does not know it: what is computed from it stays in the loop over the layers (hoisted out of it, the
// offsets of all phases took more registers than there are).
__device__ __forceinline__ int ss_fresh(int v) { asm volatile("" : "+v"(v)); return v; }
__device__ __forceinline__ float all_lanes_sum(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum_lane63(v)), 63));
}

// NR dot products per unit, units dealt to the waves of the grid workgroup first: epi(unit, sums) in lane 0.  As many of a wave's units as
// SS_CH pieces of a row hold are requested together (four rows of 256 elements, two of 512), the first ones before the vector is waited
// for: with one row at a time every further one cost a memory round trip (41.3 us a step against 36.5).  stage() brings the vector into xs
// (and ends with a barrier); false: a wait gave up.
template <int NR, typename RowPtr, typename Stage, typename Epi>
__device__ __forceinline__ bool ss_rows(int units, int K, const float* xs, RowPtr row, Stage stage, Epi epi) {
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
      for (int j = 0; j < NR; ++j) w[c][j] = *reinterpret_cast<const f32x4_t*>(row(unit, j) + min(k_of(c), K - 4));
    }
  };
  fetch();
  if (!stage()) return false;
  for (; u < units; u += together * step) {
    float s[SS_CH][NR];
    auto dot = [&](const f32x4_t& a, int k, float t) __attribute__((always_inline)) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(xs + k);
      t = fmaf(a.x, x.x, t); t = fmaf(a.y, x.y, t); t = fmaf(a.z, x.z, t);
      return fmaf(a.w, x.w, t);
    };
#pragma unroll
    for (int c = 0; c < SS_CH; ++c)
#pragma unroll
      for (int j = 0; j < NR; ++j) s[c][j] = k_of(c) < K ? dot(w[c][j], k_of(c), 0.f) : 0.f;
    for (int k = (SS_CH * 64 + lane) * 4; k < K; k += 256)
#pragma unroll
      for (int j = 0; j < NR; ++j) s[0][j] = dot(*reinterpret_cast<const f32x4_t*>(row(u, j) + k), k, s[0][j]);
    const int u0 = u;
    auto emit = [&](int unit, const float (&v)[NR]) __attribute__((always_inline)) {
      if (unit >= units) return;
      float t[NR];
#pragma unroll
      for (int j = 0; j < NR; ++j) t[j] = all_lanes_sum(v[j]);
      if (lane == 0) epi(unit, t);
    };
    auto add = [&](int a, int b) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NR; ++j) s[a][j] += s[b][j];
    };
    if (u + together * step < units) { u += together * step; fetch(); u = u0; }
    if (together == 4) {
#pragma unroll
      for (int c = 0; c < SS_CH; ++c) emit(u0 + c * step, s[c]);
    } else if (together == 2) {
      add(0, 1); emit(u0, s[0]);
      add(2, 3); emit(u0 + step, s[2]);
    } else {
      add(0, 1); add(2, 3); add(0, 2);
      emit(u0, s[0]);
    }
  }
  return true;
}

template <int HD>
__global__ void __launch_bounds__(SS_THREADS, 4) k_small_step(SmallStep P) {
  extern __shared__ __align__(16) float smem_f[];
  constexpr int HALF = HD / 2, KT = 2048 / HD;        // keys of a tile: a lane has 32 dims of one
  constexpr int VL = HD / 4, SUB = 64 / VL;          // lanes that a value row takes, value rows of a request
  const DecParams& p = P.d;
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63, wg = blockIdx.x, b = p.b;
  const int D = p.D, F = p.F, nq = p.Hq * HD, nkv = p.Hkv * HD, kmax = max(D, max(nq, F));
  float* hbuf = smem_f;                              // the residual
  float* xbuf[2] = {hbuf + D, hbuf + D + kmax};      // the vector that is multiplied, two in turn: a wave may still read the one before
  float* red[2] = {xbuf[1] + kmax, xbuf[1] + kmax + SS_WAVES};
  float* qs = red[1] + SS_WAVES;
  float *kn = qs + HD, *vn = kn + HD;
  float2* cs = reinterpret_cast<float2*>(vn + HD);
  float* parts = vn + 2 * HD;                          // [wave][HD dims, max, sum]
  Best* wbest = reinterpret_cast<Best*>(parts + SS_WAVES * (HD + 2));
  int* bad = reinterpret_cast<int*>(wbest + SS_WAVES);
  if (__hip_atomic_load(P.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1) return;
  const int pos = uni(p.len[b]), n_kept = uni(P.n_kept[b]), tok = min(max(p.tokens[b], 0), p.V - 1);
  unsigned ep = *P.epoch;
  if (ep > ~0u - (5u * n_kept + 1u)) ep = 0u;        // (five epochs a layer, one for the candidates)
  const int head = wg, g = head / p.G;               // workgroups 0 .. Hq - 1: a query head each
  const bool attends = wg < p.Hq;
  for (int i = tid; i < D; i += SS_THREADS) hbuf[i] = reinterpret_cast<const float*>(p.embed)[(size_t)tok * D + i];
  if (tid == 0) *bad = 0;
  __syncthreads();

  int turn = 0;
  float* xs = xbuf[0];
  float rms = 0.f;
  // xs = x * gain of the residual of this epoch (0, nobody's: the embedding, which is in hbuf), and what 1/rms multiplies the results with
  auto stage_norm = [&](const float* gain, unsigned epoch) __attribute__((always_inline)) {
    float ss = 0.f;
    auto take = [&](int i, float v) __attribute__((always_inline)) { hbuf[i] = v; xs[i] = v * gain[i]; ss = fmaf(v, v, ss); };
    if (epoch == 0) {
      for (int i = tid; i < D; i += SS_THREADS) take(i, hbuf[i]);
    } else if (!ss_get(P.xh, D, epoch, P.err, take)) {
      *bad = 1;
    }
    ss = all_lanes_sum(ss);
    if (lane == 0) red[turn][wave] = ss;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < SS_WAVES; ++w) t += red[turn][w];
    rms = 1.0f / sqrtf(t / (float)D + p.eps);
    return *bad == 0;
  };
  auto stage_plain = [&](const ss_word* src, int n, unsigned epoch) __attribute__((always_inline)) {
    if (!ss_get(src, n, epoch, P.err, [&](int i, float v) __attribute__((always_inline)) { xs[i] = v; })) *bad = 1;
    __syncthreads();
    return *bad == 0;
  };
  auto next = [&]() __attribute__((always_inline)) { turn ^= 1; xs = xbuf[turn]; };

  unsigned ep_h = 0;                                 // epoch of the residual that the next norm reads
  for (int kl = 0; kl < n_kept; ++kl) {
    const LayerDev l = P.layers[uni(P.kept[(size_t)b * P.L + kl])];
    const float *wq = reinterpret_cast<const float*>(l.wq), *wk = reinterpret_cast<const float*>(l.wk), *wv = reinterpret_cast<const float*>(l.wv);
    const float *wo = reinterpret_cast<const float*>(l.wo), *wd = reinterpret_cast<const float*>(l.wd);
    const float *wgt = reinterpret_cast<const float*>(l.wg), *wup = reinterpret_cast<const float*>(l.wu);
    float* pool = reinterpret_cast<float*>(l.kv);
    const unsigned e_qkv = ep + 1, e_attn = ep + 2, e_o = ep + 3, e_z = ep + 4, e_d = ep + 5;
    ep += 5;
    if (!ss_rows<1>(nq + 2 * nkv, D, xs,
                    [&](int r, int) __attribute__((always_inline)) { return r < nq ? wq + (size_t)r * D : r < nq + nkv ? wk + (size_t)(r - nq) * D : wv + (size_t)(r - nq - nkv) * D; },
                    [&]() __attribute__((always_inline)) { return stage_norm(l.g_attn, ep_h); }, [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xqkv + r, s[0] * rms, e_qkv); }))
      return;
    next();
    if (attends) {
      const size_t head_off = (size_t)g * p.P * HD, v_off = (size_t)p.Hkv * p.P * HD;
      const int* pt = p.page_table + (size_t)b * p.max_pages;
      const int ln = ss_fresh(lane), tiles = pos / KT + 1, klane = ln % KT, part = ln / KT, sub = ln / VL, vd = ln % VL;
      f32x4_t kf[8];                                 // dims 32 part .. + 32 of this lane's key
      f32x4_t vf[8];                                 // dims 4 vd .. + 4 of keys SUB i + sub
      // (keys that are not in the cache - this step's, and those behind it - are clamped to one that is, and replaced)
      auto fetch = [&](int t) __attribute__((always_inline)) {
        const int key = min(t * KT + klane, max(pos - 1, 0));
        const int off = pt[key / p.P] * (int)p.page_elems + (key % p.P) * HD;        // (a pool has fewer than 2^31 elements)
        const float* kp = pool + head_off + off + 32 * part;
#pragma unroll
        for (int c = 0; c < 8; ++c) kf[c] = *reinterpret_cast<const f32x4_t*>(kp + 4 * c);
#pragma unroll
        for (int i = 0; i < 8; ++i) vf[i] = *reinterpret_cast<const f32x4_t*>(pool + head_off + v_off + __shfl(off, SUB * i + sub, 64) + 4 * vd);
      };
      fetch(min(wave, tiles - 1));                   // (a wave without a tile loads one all the same: no branch around 64 registers)
      if (kl == 0 && tid < HALF) {                   // (behind the first projections: nobody waits for it there)
        const double a = (double)pos * p.theta[tid];
        cs[tid] = make_float2((float)cos(a), (float)sin(a));
      }
      // q, k, v of the head: qs, kn, vn raw; rotated in place behind the barrier
      const ss_word *xq = P.xqkv + head * HD, *xk = P.xqkv + nq + g * HD;
      const bool ok = ss_get_w<(3 * HD + SS_THREADS - 1) / SS_THREADS>([=](int i) __attribute__((always_inline)) { return i < HD ? xq + i : i < 2 * HD ? xk + (i - HD) : xk + (nkv + i - 2 * HD); },
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
      if (head == g * p.G && tid < HD) {             // one head of the group appends the new position
        float* dst = pool + (size_t)pt[pos / p.P] * p.page_elems + head_off + (size_t)(pos % p.P) * HD + tid;
        dst[0] = kn[tid];
        dst[v_off] = vn[tid];
      }
      float m = -INFINITY, sum = 0.f;
      f32x4_t o = {0.f, 0.f, 0.f, 0.f};
      const f32x4_t v_new = *reinterpret_cast<const f32x4_t*>(vn + 4 * vd);
      for (int t = wave; t < tiles; t += SS_WAVES) {
        const int k0 = t * KT, key = k0 + klane, d0 = 32 * ss_fresh(part);
        if (t == tiles - 1) {                        // the new position, and what is behind it (weight 0)
          if (key >= pos) {
#pragma unroll
            for (int c = 0; c < 8; ++c) kf[c] = *reinterpret_cast<const f32x4_t*>(kn + d0 + 4 * c);
          }
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
        if (HD == 128) sc += __shfl_xor(sc, 16, 64);
        sc += __shfl_xor(sc, 32, 64);
        if (key > pos) sc = -INFINITY;
        const float mn = fmaxf(m, wave_max(sc)), corr = expf(m - mn), pj = key <= pos ? expf(sc - mn) : 0.f;
        sum = sum * corr + all_lanes_sum(part == 0 ? pj : 0.f);
        m = mn;
        o *= corr;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float w = __shfl(pj, SUB * i + sub, 64);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = fmaf(w, vf[i][e], o[e]);
        }
        fetch(min(t + SS_WAVES, tiles - 1));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (SUB == 4) o[e] += __shfl_xor(o[e], 16, 64);
        o[e] += __shfl_xor(o[e], 32, 64);
        if (sub == 0) parts[wave * (HD + 2) + 4 * vd + e] = o[e];
      }
      if (lane == 0) { parts[wave * (HD + 2) + HD] = m; parts[wave * (HD + 2) + HD + 1] = sum; }
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
        ss_put(P.xattn + head * HD + tid, num / den, e_attn);
      }
    }
    if (!ss_rows<1>(D, nq, xs, [&](int r, int) __attribute__((always_inline)) { return wo + (size_t)r * nq; }, [&]() __attribute__((always_inline)) { return stage_plain(P.xattn, nq, e_attn); },
                    [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xh + r, hbuf[r] + s[0], e_o); }))
      return;
    next();
    if (!ss_rows<2>(F, D, xs, [&](int r, int j) __attribute__((always_inline)) { return (j ? wup : wgt) + (size_t)r * D; }, [&]() __attribute__((always_inline)) { return stage_norm(l.g_mlp, e_o); },
                    [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xz + r, siluf(s[0] * rms) * (s[1] * rms), e_z); }))
      return;
    next();
    if (!ss_rows<1>(D, F, xs, [&](int r, int) __attribute__((always_inline)) { return wd + (size_t)r * F; }, [&]() __attribute__((always_inline)) { return stage_plain(P.xz, F, e_z); },
                    [&](int r, const float* s) __attribute__((always_inline)) { ss_put(P.xh + r, hbuf[r] + s[0], e_d); }))
      return;
    next();
    ep_h = e_d;
  }

  // logits, and the first of the best
  Best best{-INFINITY, 0x7fffffff};
  float* lg = p.logits ? p.logits + (size_t)b * p.V : nullptr;
  const float* wl = reinterpret_cast<const float*>(p.lm_head);
  if (!ss_rows<1>(p.V, D, xs, [&](int r, int) __attribute__((always_inline)) { return wl + (size_t)r * D; }, [&]() __attribute__((always_inline)) { return stage_norm(p.g_final, ep_h); },
                  [&](int r, const float* s) __attribute__((always_inline)) {
                    const Best c{s[0] * rms, r};
                    if (lg) lg[r] = c.v;
                    if (better(c, best)) best = c;
                  }))
    return;
  ++ep;
  if (lane == 0) wbest[wave] = best;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < SS_WAVES; ++w) if (better(wbest[w], best)) best = wbest[w];
    ss_put(P.xcand + 2 * wg, best.v, ep);
    ss_put(P.xcand + 2 * wg + 1, __int_as_float(best.i), ep);
  }
  if (wg != 0) return;
  for (int i = tid; i < D; i += SS_THREADS) p.h[(size_t)b * D + i] = hbuf[i];
  const bool ok = ss_get(P.xcand, 2 * (int)gridDim.x, ep, P.err, [&](int i, float v) __attribute__((always_inline)) { xbuf[turn ^ 1][i] = v; });
  if (!ok) *bad = 1;
  __syncthreads();
  if (*bad || wave != 0) return;
  best = Best{-INFINITY, 0x7fffffff};
  for (int i = lane; i < (int)gridDim.x; i += 64) {
    const Best c{xbuf[turn ^ 1][2 * i], __float_as_int(xbuf[turn ^ 1][2 * i + 1])};
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
