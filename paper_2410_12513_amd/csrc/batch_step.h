// All layers of a decode step for up to sixteen sequences as ONE persistent kernel, a 512-thread workgroup per compute unit.
//
// What bounds such a step is HBM: every matrix of a layer that somebody keeps, once.  As five launches a layer (k_bgemv_g, k_attn_mfma_b) each
// matrix pays some 8 us of starting and draining the chip on top of its bytes.  Here the workgroups stay: the first weights of a phase are
// on their way while the phase before hands its results round.
//
// A layer is five phases: Q/K/V, attention, O, gate/up, down.  The rows of a matrix are dealt to the workgroups in units of eight (gate/up: eight rows
// of each), with the whole of K, so that nothing has to be added up across workgroups: what comes out of a workgroup is final.  Within it K is
// dealt to four pairs of waves, a streaming and a serving one: K steps (of 32) 32 p + 8 w .. + 8 of pass p to pair w.  The streaming wave keeps
// chunks of eight K steps of a 16-row tile in flight (tile order, see k_tile_weights; BS_RING chunks of 8 KB, running on into the next
// phase) and multiplies them with the activations in LDS; the serving wave brings those, a pass ahead.  A wave's loads return in order, so whoever
// waits for other workgroups must have no weights in flight.  At the end of a phase the serving waves add the four waves' sums and store the
// result.  All eight waves walk the keys in attention.
//
// What travels between workgroups are 32-bit words, each layer's at its own place: the projections [slot][row] (fp32), the activations of the
// other phases in A-operand order (bf16 high and low half in one word), squares of the residual for the norms.  Every word says by itself whether it is
// there: BS_EMPTY, a NaN that no producer stores, means not yet.  So all 32 bits of a value travel, nobody counts arrivals, and an exchange
// is one store and one load.  Activations are read by every workgroup: it polls a word of each producer coherently and fetches the rest with
// ordinary loads, which the workgroups of an XCD share through its L2; if a word is not there yet they are read again coherently.
// That is sound because a word's place is written once a launch: there are two sets, which launches take in turn, and who stores
// a word empties its twin of the other set.  So no cache of this launch can hold an older value than "empty".
//
// Attention splits long sequences; the workgroup of the first split collects the others' partial results (single-reader words: it leaves
// them empty again; their producers come back to them a layer later, behind activations that depend on what that workgroup stored since).
//
// Sequences keep their slot through all layers.  A slot whose sequence skips a layer goes through its products like the others (the tile has
// sixteen rows anyway) and is left out of attention and of the residual stream.
//
// The workgroups wait for each other, so all of them have to be on the chip: step_order.h.  The waits are bounded: polls of memory by sk_poll_give_up, those for
// the other wave of a pair by bs_inside.  One that does not get what it waits for says so in *err and to its workgroup, and nothing is made of what did
// not come: a streaming wave without its activations does not count itself done, a serving wave without all sums stores none.
//
// us a step, launches per op / this kernel, bf16, embedding and head included: 8B shape, eight layers, 16 sequences of 256 to 2048 keys 1165 / 1120 (436 MB of
// weights a layer: 61 us at the 7.1 TB/s of a large read, 112 here); four of 16384 keys, three layers 633 / 608; 3B shape, six layers, three
// sequences 572 / 540; 1B shape, four layers, 16 of 1000 keys 338 / 297; eight layers, four of 300 keys 502 / 439.  What is left above
// the bytes: about 7 us at each of a layer's five exchanges (the slowest workgroup, 3 to 5 us behind the median; the sums over the pairs; the poll; the first
// activations into LDS), each workgroup's own copy of the activations among it (at sixteen slots 1.7 MB a layer of the 8B shape, as many bytes as its weights).  Variants that
// were slower: K cut across the workgroups, with partial sums to add up (four of 16384 keys 2 % slower than launches per op, sixteen sequences 1.4 % faster
// where this is 3.9); squares of the norms polled together with the activations (b16 2 % slower: four times the words a poll reads).
#pragma once
#include "decode_batch_kernels.h"

namespace first {

constexpr int BS_THREADS = 512, BS_PAIRS = 4;
constexpr int BS_RING = 3;                            // chunks in flight per streaming wave
constexpr int BS_CHUNK = 8, BS_PASS = BS_PAIRS * BS_CHUNK;   // K steps of a chunk, of a pass
constexpr unsigned BS_EMPTY = 0xffffffffu;
constexpr int BS_MAX_L = 128, BS_WORKS = 64;          // layers; splits of all sequences for one KV head
constexpr int BS_MAX_WGS = 256;                       // (four lanes' worth of squares a slot)
constexpr int BS_OWN = 32;                            // rows of the residual stream a workgroup can own
constexpr int BS_PAGES = 256;                         // page ids of attention's item that are fetched ahead

// A phase: units of eight rows, K steps of a row.
struct BsPhase { int units, ksteps; };
struct BsLayer { const bf16 *qkv, *o, *g, *d; const float *g_attn, *g_mlp; };      // (up stands behind gate, see up_offset)

// Words of one layer: the inputs of the phases (O: attention's output), the projections, the squares of the two norm ops' inputs.
struct BsWords { unsigned in[4], squares[4], proj, all; };
__host__ __device__ inline int bs_slots(int n) { return n <= 4 ? 4 : n <= 8 ? 8 : 16; }
__host__ __device__ inline BsWords bs_words(int D, int nq, int nkv, int F, int slots, int ncu) {
  BsWords w{};
  unsigned at = 0;
  w.in[BG_QKV] = at; at += D * slots;
  w.in[BG_O] = at; at += nq * slots;
  w.in[BG_GU] = at; at += D * slots;
  w.in[BG_DN] = at; at += F * slots;
  w.proj = at; at += (nq + 2 * nkv) * slots;
  w.squares[BG_QKV] = at; at += 16 * ncu;
  w.squares[BG_GU] = at; at += 16 * ncu;
  w.all = (at + 63) / 64 * 64;
  return w;
}

struct BatchStep {
  DecParams d;                // geometry and per-sequence state (slot = sequence)
  const BsLayer* layers;
  const LayerDev* pools;      // (the layers' KV pools)
  const uint8_t* mask;        // [n][L]
  int L, n, slots;            // slots = bs_slots(n)
  BsPhase phase[4];           // BG_QKV, BG_O, BG_GU, BG_DN
  unsigned up_offset;         // bytes from a gate tile to the up tile of the same rows
  unsigned *ex, *ex_next;     // this launch's set and the other one
  unsigned* att;              // [item][G][HD + 4] partial results of attention's splits
  BsWords w;
  int x_bytes, acc_tiles, own;        // LDS: activations (and attention), sums of a wave's tiles, rows of the residual stream
  const float* g_final;
  bf16 *xh, *xl;              // input of the final norm's consumer, as k_xsplit leaves it, ...
  float* ssq_part;            // ... and its sums of squares per workgroup
  int* err;
};
__host__ __device__ inline int bs_items(int Hkv, int ncu) { return 16 * Hkv > ncu ? 16 * Hkv : ncu; }
// Most tiles of a workgroup: u units lie in this many 16-row tiles at worst (gate/up: a tile each).
__host__ __device__ inline int bs_tiles(const BsPhase& p, int ncu, bool two) {
  const int most = (p.units + ncu - 1) / ncu;
  return two ? most : p.units % ncu == 0 && most % 2 == 0 ? most / 2 : most / 2 + 1;
}
constexpr int BS_X_LDS = BS_PAIRS * 32 * 1024;        // every pair: 32 / slots passes of 1 KB a slot
__host__ __device__ inline size_t bs_lds(int x_bytes, int acc_tiles, int own) {
  return (size_t)x_bytes + (size_t)BS_PAIRS * acc_tiles * 1024 + sizeof(float) * (own * 16 + BS_MAX_L + BS_PAGES + 16 + BS_WORKS + 16 + 16 + 16);
}

__device__ __forceinline__ BatchStep bs_params() { return sk_const<BatchStep>(sk_args()); }
// What the arguments say of phase `kind`: a field of an array of them.
template <typename T>
__device__ __forceinline__ T bs_param_of(size_t array, int kind) { return sk_const<T>(sk_args() + array + kind * sizeof(T)); }
__device__ __forceinline__ BsPhase bs_phase(int kind) { return bs_param_of<BsPhase>(__builtin_offsetof(BatchStep, phase), kind); }
// Its input words in the kl-th kept layer, and their squares.
__device__ __forceinline__ unsigned* bs_input(const BatchStep& P, int kind, int kl) {
  return P.ex + (size_t)kl * P.w.all + bs_param_of<unsigned>(__builtin_offsetof(BatchStep, w.in), kind);
}
__device__ __forceinline__ unsigned* bs_squares(const BatchStep& P, int kind, int kl) {
  return P.ex + (size_t)kl * P.w.all + bs_param_of<unsigned>(__builtin_offsetof(BatchStep, w.squares), kind);
}
// What these are made of is in registers from here on (the compiler would rather load it where it is used).
template <typename T>
__device__ __forceinline__ void bs_pin1(T v) { asm volatile("" : : "s"(v)); }
template <typename... T>
__device__ __forceinline__ void bs_pin(T... v) { (bs_pin1(v), ...); }

__device__ __forceinline__ unsigned bs_word(float v) {
  const unsigned u = __float_as_uint(v);
  return u == BS_EMPTY ? 0x7fc00000u : u;
}
// bf16 high and low half of an activation in one word
__device__ __forceinline__ unsigned bs_split_word(float v) {
  const unsigned hi = pk_bf16(v, 0.f) & 0xffffu, lo = pk_bf16(v - __uint_as_float(hi << 16), 0.f) & 0xffffu, u = (hi << 16) | lo;
  return u == BS_EMPTY ? 0xffff0000u : u;
}
__device__ __forceinline__ void bs_st(unsigned* p, unsigned v) { __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ unsigned bs_ld(const unsigned* p) { return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Stores a word of the exchange and empties its twin.
__device__ __forceinline__ void bs_put(const BatchStep& P, unsigned* p, unsigned v) {
  bs_st(p, v);
  *as_global(P.ex_next + (p - P.ex)) = BS_EMPTY;
}
// The largest of the words: BS_EMPTY exactly if one of them is.
__device__ __forceinline__ unsigned bs_most(const u32x4_t& a, unsigned m) { return max(max(max(a.x, a.y), max(a.z, a.w)), m); }
using BsCached = std::integral_constant<int, 0>;
using BsCoherent = std::integral_constant<int, 17>;   // sc0 sc1

// ready() until it holds in every lane; false: gave up.
template <typename F>
__device__ __forceinline__ bool bs_poll(int* err, F ready) {
  unsigned spins = 0;
  for (;;) {
    const int e = (int)bs_ld(reinterpret_cast<unsigned*>(err));
    const bool ok = ready();
    if (__all(ok)) { asm volatile("" ::: "memory"); return true; }
    if (sk_poll_give_up(spins, uni(e), err)) return false;
  }
}
// 16 bytes a lane from (descriptor base + voff + soff) to LDS byte lds_off + 16 * lane.  No vector register is written; bs_wait_loads orders it.
// (The LDS offset travels in m0, as an operand: the compiler writes the register, so it knows.)
typedef int i32x4_bs __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void bs_load_lds(unsigned lds_off, unsigned voff, i32x4_bs rsrc, unsigned soff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// Waits until at most n of this wave's memory operations are on their way (n: a multiple of four below 32).
__device__ __forceinline__ void bs_wait_loads(int n) {
  switch (n >> 2) {
    case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(12)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(16)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(20)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(24)" ::: "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(28)" ::: "memory"); break;
  }
}
// A counter in LDS that waves of this workgroup advance.
__device__ __forceinline__ int bs_count(const int* c) { return uni(__hip_atomic_load(c, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)); }

// Until there() holds, which another wave of this workgroup sees to; false: it never will.
template <typename F>
__device__ __forceinline__ bool bs_inside(int* bad, int* err, F there) {
  const WaitEnd end = wait_inside(there, [=]() __attribute__((always_inline)) { return bs_count(bad) != 0; }, []() __attribute__((always_inline)) { __builtin_amdgcn_s_sleep(1); });
  if (end == WaitEnd::RAN_OUT) {
    *bad = 1;
    __hip_atomic_fetch_or(as_global(err), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return end == WaitEnd::THERE;
}

// Empties the first n words of both sets and attention's.
__global__ void __launch_bounds__(WG) k_empty_words(unsigned* ex, unsigned* ex2, size_t n, unsigned* att, size_t n_att) {
  for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n; i += (size_t)gridDim.x * WG) { ex[i] = BS_EMPTY; ex2[i] = BS_EMPTY; }
  for (size_t i = (size_t)blockIdx.x * WG + threadIdx.x; i < n_att; i += (size_t)gridDim.x * WG) att[i] = BS_EMPTY;
}

// A workgroup's share of a phase: units [u0, u1) and the 16-row tiles they lie in (gate/up: a unit is a tile, eight rows of each matrix).
struct BsShare { int u0, u1, tile0, tiles; };
__device__ __forceinline__ BsShare bs_share(const BsPhase& ph, bool two) {
  const unsigned wg = blockIdx.x, ncu = gridDim.x;
  BsShare s;
  s.u0 = (int)((unsigned)ph.units * wg / ncu); s.u1 = (int)((unsigned)ph.units * (wg + 1) / ncu);
  s.tile0 = two ? s.u0 : s.u0 >> 1;
  s.tiles = two ? s.u1 - s.u0 : s.u1 > s.u0 ? ((s.u1 + 1) >> 1) - s.tile0 : 0;
  return s;
}

// A streaming wave's weights of a phase: chunk (p, t) = eight K steps of the workgroup's t-th tile in pass p.
struct BsSeg { unsigned long long m; int u0, u1, tile0, tiles, passes, ksteps, two; };
__device__ __forceinline__ BsSeg bs_seg(const BatchStep& P, int kind, int layer, int wave) {
  const BsPhase ph = bs_phase(kind);
  const BsShare sh = bs_share(ph, kind == BG_GU);
  // the matrices stand in the table in the order of the phases
  BsSeg s;
  s.m = sk_const<unsigned long long>(reinterpret_cast<unsigned long long>(P.layers) + layer * sizeof(BsLayer) + 8 * kind);
  s.u0 = uni(sh.u0); s.u1 = uni(sh.u1); s.tile0 = uni(sh.tile0); s.tiles = uni(sh.tiles);
  s.ksteps = ph.ksteps; s.two = kind == BG_GU;
  s.passes = s.tiles > 0 ? uni((ph.ksteps / BS_CHUNK - wave + BS_PAIRS - 1) / BS_PAIRS) : 0;
  return s;
}
// Requests chunk (p, t): 1 KB a K step.  Rows that belong to another workgroup, and chunks that do not exist, lie beyond the descriptor: zeros, and
// no access.
__device__ __forceinline__ void bs_issue(const BsSeg& s, int p, int t, int wave, int lane, unsigned up_offset, u32x4_t (&b)[BS_CHUNK]) {
  const int tile = s.tile0 + t, k = p * BS_PASS + wave * BS_CHUNK;
  const unsigned long long a = sk_uniform(s.m + (((unsigned long long)(unsigned)(s.two ? tile >> 1 : tile) * (unsigned)s.ksteps + (unsigned)k) << 10));
  const __amdgpu_buffer_rsrc_t d0 = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(a), (short)0, uni(p < s.passes ? 0x7fffffff : 0), 0x00020000);
  const __amdgpu_buffer_rsrc_t d1 = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(a + 4096), (short)0, uni(p < s.passes ? 0x7fffffff : 0), 0x00020000);
  const int half = (lane >> 3) & 1;                   // of the tile's rows
  unsigned off;
  if (s.two) {                                        // lanes of the lower rows: gate, of the upper ones: up - rows 8 (tile & 1) .. + 8 of both
    off = (unsigned)((lane & 0x37) | ((tile & 1) << 3)) * 16u + (half ? up_offset : 0u);
  } else {
    const int u = 2 * tile + half;
    off = u >= s.u0 && u < s.u1 ? (unsigned)lane * 16u : 0x80000000u;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) b[u] = __builtin_amdgcn_raw_buffer_load_b128(d0, off + u * 1024, 0, 2);          // 2 = non-temporal
#pragma unroll
  for (int u = 0; u < 4; ++u) b[4 + u] = __builtin_amdgcn_raw_buffer_load_b128(d1, off + u * 1024, 0, 2);
}

// Streams phase `cur`, whose first BS_RING chunks are in the ring, and requests the first ones of `nxt` behind it.  x: this pair's activations, two
// passes in turn; acc: this wave's sums, [tile][lane].  One code for all phases.
struct BsLink { int* staged; int* consumed; int* done; int* bad; int base, n; const unsigned* words; int* err; };     // counters in LDS: passes staged / taken so far, base at the phase's start
__device__ __forceinline__ void bs_stream(const BsSeg& cur, const BsSeg& nxt, u32x4_t (&ring)[BS_RING][BS_CHUNK], const char* x, int slots, f32x4_t* acc, unsigned up_offset, int wave,
                                          const BsLink& link) {
  const int lane = sk_lane_opaque();
  const int total = cur.passes * cur.tiles, padded = max(BS_RING, (total + BS_RING - 1) / BS_RING * BS_RING);
  const int ring_mask = 32 / slots - 1;               // passes in LDS
  const int place = ((lane >> 4) * slots + min(lane & 15, slots - 1)) * 32;      // of this lane's eight words of a K step
  const bool live = (lane & 15) < link.n;
  u32x4_t ah[BS_CHUNK], al[BS_CHUNK];                 // the pass's activations, for all its tiles
  auto split = [&](int u, const u32x4_t& a, const u32x4_t& b) __attribute__((always_inline)) {
    ah[u].x = __builtin_amdgcn_perm(a.y, a.x, 0x07060302); ah[u].y = __builtin_amdgcn_perm(a.w, a.z, 0x07060302);
    ah[u].z = __builtin_amdgcn_perm(b.y, b.x, 0x07060302); ah[u].w = __builtin_amdgcn_perm(b.w, b.z, 0x07060302);
    al[u].x = __builtin_amdgcn_perm(a.y, a.x, 0x05040100); al[u].y = __builtin_amdgcn_perm(a.w, a.z, 0x05040100);
    al[u].z = __builtin_amdgcn_perm(b.y, b.x, 0x05040100); al[u].w = __builtin_amdgcn_perm(b.w, b.z, 0x05040100);
  };
  int cp = 0, ct = 0;                                 // pass and tile that is multiplied next
  int rp = 0, rt = 0;                                 // ... that is requested next
  auto step = [](int& p, int& t, int tiles) __attribute__((always_inline)) { if (++t >= tiles) { t = 0; ++p; } };
  for (int j = 0; j < BS_RING; ++j) step(rp, rt, cur.tiles);
  auto consume = [&](const u32x4_t (&b)[BS_CHUNK]) __attribute__((always_inline)) {
    if (ct == 0) {
      // (without its activations the wave walks through the rest on what is in LDS, waits for nothing - whoever has set *bad has set *err - and does not
      // count itself done: a branch here would make two kernels of this one, with 34 registers more)
      bs_inside(link.bad, link.err, [&]() __attribute__((always_inline)) { return bs_count(link.staged) > link.base + cp; });
      const char* xc = x + (cp & ring_mask) * slots * 1024 + place;
      unsigned most = 0;
#pragma unroll
      for (int h = 0; h < BS_CHUNK; h += 4) {
        u32x4_t a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const char* at = xc + (h + u) * slots * 128;
          a[u] = *reinterpret_cast<const u32x4_t*>(at);
          b[u] = *reinterpret_cast<const u32x4_t*>(at + 16);
        }
        __builtin_amdgcn_sched_barrier(0);            // (requested together: left alone, the compiler fetches them one by one and waits for each)
#pragma unroll
        for (int u = 0; u < 4; ++u) { most = bs_most(b[u], bs_most(a[u], most)); split(h + u, a[u], b[u]); }
      }
      if (lane == 0) __hip_atomic_store(link.consumed, link.base + cp + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (!__all(most != BS_EMPTY || !live)) {        // a word was not there yet although its producer's first one was: read the pass itself, coherently
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned*>(uni(link.words)), (short)0, cur.ksteps * slots * 128, 0x00020000);
        if (!bs_poll(link.err, [&]() __attribute__((always_inline)) {
          unsigned m = 0;
#pragma unroll
          for (int u = 0; u < BS_CHUNK; ++u) {
            const int at = (cp * BS_PASS + wave * BS_CHUNK + u) * slots * 128 + place;
            const u32x4_t a = __builtin_amdgcn_raw_buffer_load_b128(rs, at, 0, BsCoherent::value), b = __builtin_amdgcn_raw_buffer_load_b128(rs, at + 16, 0, BsCoherent::value);
            m = bs_most(b, bs_most(a, m));
            split(u, a, b);
          }
          return m != BS_EMPTY || !live;
        })) *link.bad = 1;
      }
    }
    f32x4v_t hi = {0.f, 0.f, 0.f, 0.f}, lo = {0.f, 0.f, 0.f, 0.f};
    if (cp > 0) { const f32x4_t was = acc[ct * 64 + lane]; hi = f32x4v_t{was.x, was.y, was.z, was.w}; }
#pragma unroll
    for (int u = 0; u < BS_CHUNK; ++u) {
      hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ah[u]), as_bf16x8(b[u]), hi, 0, 0, 0);
      lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(al[u]), as_bf16x8(b[u]), lo, 0, 0, 0);
    }
    acc[ct * 64 + lane] = f32x4_t{hi[0] + lo[0], hi[1] + lo[1], hi[2] + lo[2], hi[3] + lo[3]};
    step(cp, ct, cur.tiles);
  };
  for (int c0 = 0; c0 < padded; c0 += BS_RING) {
    BsSeg g = cur;
    if (c0 + BS_RING >= padded) { g = nxt; rp = 0; rt = 0; }
#pragma unroll
    for (int j = 0; j < BS_RING; ++j) {
      if (c0 + j < total) consume(ring[j]);
      if (c0 + j == max(total, 1) - 1 && bs_count(link.bad) == 0 && lane == 0) __hip_atomic_fetch_add(link.done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      bs_issue(g, rp, rt, wave, lane, up_offset, ring[j]);
      step(rp, rt, g.tiles);
    }
  }
}

// This step's projections of one KV head and one sequence.
template <int HD, int G>
struct BsQkv {
  const unsigned* proj;                               // of this slot
  int* err;
  float* raw;                                         // LDS: G queries, key, value
  int* bad;
  int* pages;                                         // LDS: the split's first BS_PAGES page ids, where they have been fetched ahead
  int g, Hkv;
  __device__ __forceinline__ int* ahead(int n) const { return n <= BS_PAGES ? pages : nullptr; }
  __device__ __forceinline__ void request(int, int, int, int) {}
  __device__ __forceinline__ void arrive() {
    constexpr int N = (G + 2) * HD, R = (N + BS_THREADS - 1) / BS_THREADS;
    const int tid = uni((int)(threadIdx.x >> 6)) * 64 + sk_lane_opaque();
    unsigned w[R];
    if (!bs_poll(err, [&]() __attribute__((always_inline)) {
          unsigned m = 0;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int e = min(tid + r * BS_THREADS, N - 1);
            w[r] = bs_ld(proj + (e < G * HD ? g * G * HD + e : Hkv * G * HD + (e < (G + 1) * HD ? g * HD + (e - G * HD) : (Hkv + g) * HD + (e - (G + 1) * HD))));
          }
#pragma unroll
          for (int r = 0; r < R; ++r) m = max(m, w[r]);
          return m != BS_EMPTY;
        }))
      *bad = 1;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * BS_THREADS < N) raw[tid + r * BS_THREADS] = __uint_as_float(w[r]);
  }
  __device__ __forceinline__ void get(float& q1, float& q2, float& k1, float& k2, float& v, int iq, int dk, int dv, int half) {
    q1 = raw[iq]; q2 = raw[iq + half];
    k1 = raw[G * HD + dk]; k2 = raw[G * HD + dk + half];
    v = raw[(G + 1) * HD + dv];
  }
};
__host__ __device__ inline size_t bs_attn_lds(int G, int hd) { return as_lds_bytes(G, hd) + (size_t)(G + 2) * hd * sizeof(float); }

template <int HD, int G>
__global__ void __launch_bounds__(BS_THREADS) k_batch_step(BatchStep) {
  extern __shared__ __align__(16) unsigned char smem_b[];
  const int tid = threadIdx.x, wave = uni(tid >> 6), wg = blockIdx.x, ncu = gridDim.x;
  const int n = uni(bs_params().n), slots = uni(bs_params().slots);
  f32x4_t* acc = reinterpret_cast<f32x4_t*>(smem_b + bs_params().x_bytes);     // [pair][tile][64]
  const int acc_pair = uni(bs_params().acc_tiles) * 64;
  float* hl = reinterpret_cast<float*>(acc + BS_PAIRS * acc_pair);     // this workgroup's rows of the residual stream, [row][16]
  int* kept = reinterpret_cast<int*>(hl + bs_params().own * 16);        // layer | sequences that keep it << 16
  int* pages = kept + BS_MAX_L;                                 // of this workgroup's item of attention
  int* pos = pages + BS_PAGES;
  int* works = pos + 16;                                        // attention: slot | split << 8, in the order of the slots
  int* wcnt = works + BS_WORKS;                                 // a slot's splits
  float* rinv = reinterpret_cast<float*>(wcnt + 16);
  int* ctl = reinterpret_cast<int*>(rinv + 16);
  int *bad = ctl, *done = ctl + 1, *n_works = ctl + 2, *n_kept = ctl + 3, *staged = ctl + 4, *consumed = ctl + 8;
  if (wave == 0) {                                              // layers that somebody keeps
    const BatchStep P = bs_params();
    const int gave_up = (int)bs_ld(reinterpret_cast<const unsigned*>(P.err)) & 1;      // in an earlier launch: its words are in nobody's order
    const int L = P.L, lane = tid & 63;
    const uint8_t* mask = P.mask;
    int nk = 0;
    for (int i0 = 0; i0 < L; i0 += 64) {
      const int i = i0 + lane;
      unsigned bits = 0;
      if (i < L)
        for (int j = 0; j < n; ++j) bits |= (*as_global(mask + (size_t)j * L + i) ? 1u : 0u) << j;
      const unsigned long long m = __ballot(bits != 0);
      if (bits) kept[nk + __popcll(m & ((1ull << lane) - 1))] = i | (int)(bits << 16);
      nk += __popcll(m);
    }
    if (lane < 12) ctl[lane] = lane == 3 ? nk : lane == 0 ? gave_up : 0;
  } else if (wave == 2) {                                       // the tables into the scalar cache, which nothing else of this kernel fills: a first look at an entry costs 2 us
    const BatchStep P = bs_params();
    unsigned seen = 0;
    for (int i = 0; i < P.L; ++i) seen |= sk_const<unsigned>(reinterpret_cast<unsigned long long>(P.layers + i)) | sk_const<unsigned>(reinterpret_cast<unsigned long long>(P.pools + i) + sizeof(LayerDev) - 8);
    asm volatile("" : : "s"(seen));
  }
  if (wave == 1 && (tid & 63) < 16) pos[tid & 63] = *as_global(bs_params().d.len + min(tid & 63, n - 1));
  lds_barrier();
  if (uni(*bad)) return;
  const int nk = uni(*n_kept);
  auto layer_of = [&](int kl) __attribute__((always_inline)) { return uni(kept[min(kl, nk - 1)] & 0xffff); };
  auto table = [&](const BatchStep& P, int layer) __attribute__((always_inline)) { return sk_const<BsLayer>(reinterpret_cast<unsigned long long>(P.layers) + layer * sizeof(BsLayer)); };
  const bool streams = wave < BS_PAIRS;
  const int pair = wave & (BS_PAIRS - 1);
  char* x = reinterpret_cast<char*>(smem_b) + pair * (BS_X_LDS / BS_PAIRS);       // this pair's activations: 32 / slots passes of high and low halves
  int base = 0;                                                 // passes of this pair in the phases before

  // ---- serving waves.  All activation words of this pair's K steps, pass by pass into LDS.
  // meanwhile(): what else there is to do, once `when` passes are there.
  auto stage = [&](const BatchStep& P, const unsigned* words, int ksteps, int passes, int when, auto meanwhile) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque();
    {                                                           // a word of each producer (they store eight rows of all slots): lane = (K step, octet) of a pass
      const int ln = lane & 31;
      if (!bs_poll(P.err, [&]() __attribute__((always_inline)) {
            unsigned m = 0;
            for (int p = lane >> 5; p < passes; p += 8) {
              unsigned w[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) w[u] = bs_ld(words + ((size_t)((min(p + 2 * u, passes - 1) * BS_PASS + pair * BS_CHUNK) * 4 + ln) * slots + min(ln & 3, n - 1)) * 8);
#pragma unroll
              for (int u = 0; u < 4; ++u) m = max(m, w[u]);
            }
            return m != BS_EMPTY;
          })) { *bad = 1; return; }
    }
    // straight into LDS, as many passes ahead as have room there (32 KB: 32 / slots, each `slots` loads of 1 KB)
    const int room = 32 / slots;
    const unsigned long long base_at = sk_uniform(reinterpret_cast<unsigned long long>(words));
    const i32x4_bs rs = {(int)(unsigned)base_at, (int)((unsigned)(base_at >> 32) & 0xffffu), uni(ksteps * slots * 128), 0x00020000};
    const unsigned x_off = (unsigned)uni((int)(unsigned)(size_t)(__attribute__((address_space(3))) void*)x);
    int issued = 0, out = 0;
    bool ahead = false;
    while (out < passes || !ahead) {
      if (!ahead && out == min(passes, when)) {
        meanwhile();
        ahead = true;
      } else if (issued < passes && bs_count(consumed + pair) >= base + issued - room + 1) {
        const unsigned lds = x_off + (unsigned)((issued & (room - 1)) * slots * 1024), from = (unsigned)((issued * BS_PASS + pair * BS_CHUNK) * slots * 128);
        for (int i = 0; i < slots; i += 4) {
#pragma unroll
          for (int u = 0; u < 4; ++u) bs_load_lds((unsigned)uni((int)(lds + (unsigned)(i + u) * 1024u)), (unsigned)lane * 16u, rs, (unsigned)uni((int)(from + (unsigned)(i + u) * 1024u)));
        }
        ++issued;
      } else if (out < issued) {
        bs_wait_loads((issued - 1 - out) * slots);
        ++out;
        if (lane == 0) __hip_atomic_store(staged + pair, base + out, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      } else if (!bs_inside(bad, P.err, [&]() __attribute__((always_inline)) { return bs_count(consumed + pair) >= base + issued - room + 1; })) {
        return;
      }
    }
  };

  // 1 / rms of this wave's slots pair, pair + 4, .. from all workgroups' squares (fixed order)
  auto norms = [&](const BatchStep& P, const unsigned* squares) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), D = P.d.D, parts = min(ncu, D >> 3);         // (of the workgroups that have a unit)
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned*>(uni(squares)), (short)0, ncu * 64, 0x00020000);
    u32x4_t w[4];
    if (!bs_poll(P.err, [&]() __attribute__((always_inline)) {
          unsigned m = 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (pair * ncu + min(u * 64 + lane, parts - 1)) * 16, 0, BsCoherent::value);
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) m = pair + 4 * j < n ? max(m, w[u][j]) : m;
          return m != BS_EMPTY;
        })) { *bad = 1; return; }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] += u * 64 + lane < parts ? __uint_as_float(w[u][j]) : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = wave_sum(s[j]);
    const float t = lane == 0 ? s[0] : lane == 1 ? s[1] : lane == 2 ? s[2] : s[3];
    if (lane < 4) rinv[pair + 4 * lane] = 1.0f / sqrtf(t / (float)D + P.d.eps);
  };

  // Sum of the four waves for element (row lane % 16, slot 4 (lane / 16) + pair) of the workgroup's t-th tile.
  auto sum = [&](int t, int lane, int ksteps) __attribute__((always_inline)) {
    const float* at = reinterpret_cast<const float*>(acc + t * 64 + lane) + pair;
    float s = at[0];
#pragma unroll
    for (int w = 1; w < BS_PAIRS; ++w) s += ksteps > w * BS_CHUNK ? at[w * acc_pair * 4] : 0.f;      // (a short row leaves pairs without a share)
    return s;
  };

  // rows of this workgroup: residual += the phase's sums (first: the residual itself, from the embedding), and what the next norm op
  // needs of it: words xw and squares sw, or behind the last layer (null) what the head reads
  // gains of this lane's rows: tile after tile (at most BS_OWN rows, in up to three tiles)
  struct Gains { float g[BS_OWN / 16 + 1]; };
  auto gains_of = [&](const BatchStep& P, const float* gain) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), D = P.d.D;
    const BsShare sh = bs_share(BsPhase{D >> 3, 0}, false);
    Gains r;
#pragma unroll
    for (int t = 0; t < BS_OWN / 16 + 1; ++t) r.g[t] = ldg(gain + min((sh.tile0 + t) * 16 + (lane & 15), D - 1));
    return r;
  };
  auto residual = [&](const BatchStep& P, bool first, int ksteps, const Gains& gains, unsigned bits, unsigned* xw, unsigned* sw) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), row16 = lane & 15, slot = 4 * (lane >> 4) + pair, D = P.d.D;
    const BsShare sh = bs_share(BsPhase{D >> 3, 0}, false);
    float sq = 0.f;
#pragma unroll
    for (int t = 0; t < BS_OWN / 16 + 1; ++t) {
      if (t >= sh.tiles) break;
      const int row = (sh.tile0 + t) * 16 + row16, u = row >> 3;
      const bool mine = u >= sh.u0 && u < sh.u1 && slot < n;
      float* keep = hl + (max(min(row - 8 * sh.u0, BS_OWN - 1), 0)) * 16 + slot;
      float h = 0.f;
      const float gn = gains.g[t];
      if (first) {
        if (mine) h = ldg(P.d.h + (size_t)slot * D + row);
      } else {
        h = *keep;
        if ((bits >> slot) & 1) h += sum(t, lane, ksteps);
      }
      if (mine) {
        *keep = h;
        sq = fmaf(h, h, sq);
        const unsigned v = bs_split_word(h * gn);
        if (xw != nullptr) {
          bs_put(P, xw + ((row >> 3) * slots + slot) * 8 + (row & 7), v);
        } else {
          const size_t to = bg_aidx(slot, row);
          stg_bf16(P.xh + to, bf16{(uint16_t)(v >> 16)});
          stg_bf16(P.xl + to, bf16{(uint16_t)v});
          *as_global(P.d.h + (size_t)slot * D + row) = h;
        }
      }
    }
    // the rows' squares: sixteen lanes of a slot
    sq = dpp_add<0xB1, 0xf>(sq); sq = dpp_add<0x4E, 0xf>(sq); sq = dpp_add<0x141, 0xf>(sq); sq = dpp_add<0x140, 0xf>(sq);
    if (row16 == 0 && sh.tiles > 0) {
      const int part = (D >> 3) >= ncu ? wg : sh.u0;
      if (xw == nullptr) *as_global(P.ssq_part + part * 16 + slot) = sq;
      else if (slot < n) bs_put(P, sw + (pair * ncu + part) * 4 + (slot >> 2), bs_word(sq));
    }
  };

  // the projections, scaled by 1 / rms
  auto projections = [&](const BatchStep& P, unsigned* proj) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), row16 = lane & 15, slot = 4 * (lane >> 4) + pair, N = P.phase[BG_QKV].units * 8;
    const BsShare sh = bs_share(P.phase[BG_QKV], false);
    for (int t = 0; t < sh.tiles; ++t) {
      const int row = (sh.tile0 + t) * 16 + row16, u = row >> 3;
      if (u >= sh.u0 && u < sh.u1 && slot < n) bs_put(P, proj + slot * N + row, bs_word(sum(t, lane, P.phase[BG_QKV].ksteps) * rinv[slot]));
    }
  };

  // z = silu(gate) * up: gate rows in the lower lanes, up in the upper ones
  auto glu = [&](const BatchStep& P, unsigned* z) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), row16 = lane & 15, slot = 4 * (lane >> 4) + pair;
    const BsShare sh = bs_share(P.phase[BG_GU], true);
    const float r = rinv[slot];
    for (int t = 0; t < sh.tiles; ++t) {
      const float v = sum(t, lane, P.phase[BG_GU].ksteps) * r, up = __shfl_xor(v, 8, 64);
      if (row16 < 8 && slot < n) bs_put(P, z + ((sh.u0 + t) * slots + slot) * 8 + row16, bs_split_word(siluf(v) * up));
    }
  };

  // splits of the sequences that keep this layer: the fewest tiles a workgroup for which one round of the chip holds them all
  auto share_out = [&](const BatchStep& P, unsigned bits) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque();
    const int tiles = lane < 16 && ((bits >> lane) & 1) ? (pos[lane & 15] + 64) >> 6 : 0;
    const int room = max(__popc(bits & 0xffffu), min(BS_WORKS, ncu / P.d.Hkv)), least = (4 * tiles + AS_PT - 1) / AS_PT;
    auto splits = [&](int tpw) __attribute__((always_inline)) { return tiles == 0 ? 0 : min(min(S_MAX, (tiles + AS_NT - 1) / AS_NT), max(least, tiles <= 10 ? 1 : (tiles + tpw - 1) / tpw)); };
    int lo_t = AS_NT, hi_t = AS_PT / 4;
    while (lo_t < hi_t) {
      const int mid = (lo_t + hi_t) >> 1;
      int total = splits(mid);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) total += __shfl_xor(total, o, 64);
      if (uni(total) <= room) hi_t = mid; else lo_t = mid + 1;
    }
    const int mine = splits(hi_t);
    int before = mine;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) { const int v = __shfl_up(before, o, 64); if (lane >= o) before += v; }
    if (lane < 16) {
      wcnt[lane] = mine;
      for (int q = 0; q < mine; ++q) works[before - mine + q] = lane | (q << 8);
      if (lane == 15) *n_works = before;
    }
  };

  // page ids of this workgroup's first item (by the wave that has just shared them out)
  auto fetch_pages = [&](const BatchStep& P) __attribute__((always_inline)) {
    const int lane = sk_lane_opaque(), w = (int)((unsigned)wg / (unsigned)P.d.Hkv);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (w >= uni(*n_works)) return;
    const int wk = uni(works[w]), slot = wk & 0xff, at = uni(pos[slot]), tiles = (at + 64) >> 6, tps = (tiles + wcnt[slot] - 1) / wcnt[slot];
    const int count = min(min(tps, tiles - (wk >> 8) * tps) * 4, BS_PAGES);
    const int* pt = P.d.page_table + (size_t)slot * P.d.max_pages;
    for (int i = lane; i < count; i += 64) pages[i] = *as_global(pt + min((wk >> 8) * tps * 4 + i, at / P.d.P));
  };

  u32x4_t ring[BS_RING][BS_CHUNK];                                // (of a streaming wave)
  BsSeg cur;
  // (a serving wave has none: without a word the compiler would keep those registers for it through everything it does)
  auto no_ring = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < BS_RING; ++j)
#pragma unroll
      for (int u = 0; u < BS_CHUNK; ++u) asm volatile("" : "=v"(ring[j][u]));
  };
  auto first_chunks = [&](unsigned up_offset) __attribute__((always_inline)) {
    int p = 0, t = 0;
    const int lane = sk_lane_opaque();
#pragma unroll
    for (int j = 0; j < BS_RING; ++j) {
      bs_issue(cur, p, t, pair, lane, up_offset, ring[j]);
      if (++t >= cur.tiles) { t = 0; ++p; }
    }
  };
  if (streams) {
    const BatchStep P = bs_params();
    cur = bs_seg(P, BG_QKV, layer_of(0), pair);
    first_chunks(P.up_offset);
  } else {
    const BatchStep P = bs_params();
    no_ring();
    residual(P, true, 0, gains_of(P, table(P, layer_of(0)).g_attn), 0, bs_input(P, BG_QKV, 0), bs_squares(P, BG_QKV, 0));
    if (pair == 0) { share_out(P, (unsigned)uni(kept[0]) >> 16); fetch_pages(P); }
  }
  for (int s = 0; s < 4 * nk; ++s) {
    const int kind = s & 3, kl = s >> 2;
    if (streams) {
      const BatchStep P = bs_params();
      BsSeg nxt = bs_seg(P, (s + 1) & 3, layer_of((s + 1) >> 2), pair);
      if (kind == BG_QKV || s + 1 == 4 * nk) nxt.passes = 0;      // (attention takes the ring's registers)
      const unsigned up_offset = P.up_offset;
      bs_pin(nxt.m, up_offset);
      bs_stream(cur, nxt, ring, x, slots, acc + pair * acc_pair, up_offset, pair, BsLink{staged + pair, consumed + pair, done, bad, base, n, bs_input(P, kind, kl), P.err});
      base += cur.passes;
      cur = nxt;
    } else {
      const BatchStep P = bs_params();
      const unsigned bits = (unsigned)uni(kept[kl]) >> 16;
      const BsPhase ph = bs_phase(kind);
      const bool dn = kind == BG_DN, last = s + 1 == 4 * nk;
      // what the phase's end needs is on its way from the start: its gains, the page ids of attention
      const BsLayer l = table(P, layer_of(dn ? kl + 1 : kl));
      const Gains gains = kind == BG_O || dn ? gains_of(P, last ? P.g_final : dn ? l.g_attn : l.g_mlp) : Gains{};
      unsigned* to = kind == BG_QKV ? P.ex + (size_t)kl * P.w.all + P.w.proj : bs_input(P, dn ? BG_QKV : kind == BG_O ? BG_GU : BG_DN, dn ? kl + 1 : kl);
      unsigned* sq = bs_squares(P, dn ? BG_QKV : BG_GU, dn ? kl + 1 : kl);
      auto meanwhile = [&]() __attribute__((always_inline)) {
        if (kind == BG_QKV || kind == BG_GU) norms(P, bs_squares(P, kind, kl));
        if (kind == BG_GU && pair == 0 && kl + 1 < nk) { share_out(P, (unsigned)uni(kept[kl + 1]) >> 16); fetch_pages(P); }
      };
      // (without a tile in this workgroup its streaming waves take nothing)
      const int passes = bs_share(ph, kind == BG_GU).tiles > 0 ? (ph.ksteps / BS_CHUNK - pair + BS_PAIRS - 1) / BS_PAIRS : 0;
      stage(P, bs_input(P, kind, kl), ph.ksteps, passes, kind == BG_GU ? 1 : passes, meanwhile);
      base += passes;
      // (a wait of this wave that gave up, for activations or squares, has set *bad)
      if (bs_inside(bad, P.err, [&]() __attribute__((always_inline)) { return bs_count(done) >= BS_PAIRS * (s + 1); }) && bs_count(bad) == 0) {
        if (kind == BG_QKV) projections(P, to);
        else if (kind == BG_GU) glu(P, to);
        else residual(P, false, ph.ksteps, gains, bits, last ? nullptr : to, sq);
      }
    }
    lds_barrier();                                                // phase over: its sums have been read
    if (uni(*bad)) return;
    if (kind == BG_QKV) {
      const BatchStep P = bs_params();
      unsigned* out = bs_input(P, BG_O, kl);
      DecParams p = P.d;
      p.kv_layer = sk_const<LayerDev>(reinterpret_cast<unsigned long long>(P.pools) + layer_of(kl) * sizeof(LayerDev)).kv;
      const int items = uni(*n_works) * p.Hkv, N = P.phase[BG_QKV].units * 8;
      for (int it = wg; it < items; it += ncu) {
        const int w = (int)((unsigned)it / (unsigned)p.Hkv), wk = uni(works[w]), g = it - w * p.Hkv, slot = wk & 0xff, split = wk >> 8, splits = uni(wcnt[slot]);
        BsQkv<HD, G> src{P.ex + (size_t)kl * P.w.all + P.w.proj + slot * N, P.err, reinterpret_cast<float*>(smem_b + as_lds_bytes(G, HD)), bad, it == wg ? pages : nullptr, g, p.Hkv};
        attn_mfma_split<HD, G>(p, slot, g, split, splits, uni(pos[slot]), reinterpret_cast<float*>(smem_b), src,
                               [&](int hq, float M, float den, float a0, float a1) __attribute__((always_inline)) {
          const int lane = sk_lane_opaque();
          unsigned* part = P.att + ((size_t)it * G + hq) * (HD + 4);
          if (split != 0) {                                       // left for the first split's workgroup
            bs_st(part + lane, bs_word(a0));
            if (HD > 64) bs_st(part + 64 + lane, bs_word(a1));
            if (lane < 2) bs_st(part + HD + lane, bs_word(lane ? den : M));
            return;
          }
          for (int q0 = 1; q0 < splits; q0 += 4) {                // ... which merges them in order
            unsigned v0[4], v1[4], vm[4], vl[4];
            if (!bs_poll(P.err, [&]() __attribute__((always_inline)) {
                  unsigned m = 0;
#pragma unroll
                  for (int u = 0; u < 4; ++u) {
                    const unsigned* at = part + (size_t)min(q0 + u, splits - 1) * p.Hkv * G * (HD + 4);
                    v0[u] = bs_ld(at + lane); v1[u] = HD > 64 ? bs_ld(at + 64 + lane) : 0; vm[u] = bs_ld(at + HD); vl[u] = bs_ld(at + HD + 1);
                  }
#pragma unroll
                  for (int u = 0; u < 4; ++u) m = max(m, max(max(v0[u], v1[u]), max(vm[u], vl[u])));
                  return m != BS_EMPTY;
                })) { *bad = 1; return; }
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (q0 + u < splits) {
                unsigned* at = part + (size_t)(q0 + u) * p.Hkv * G * (HD + 4);
                bs_st(at + lane, BS_EMPTY);
                if (HD > 64) bs_st(at + 64 + lane, BS_EMPTY);
                if (lane < 2) bs_st(at + HD + lane, BS_EMPTY);
                if (__uint_as_float(vl[u]) > 0.f) {
                  const float M2 = fmaxf(M, __uint_as_float(vm[u])), c0 = expf(M - M2), c1 = expf(__uint_as_float(vm[u]) - M2);
                  M = M2;
                  den = fmaf(den, c0, __uint_as_float(vl[u]) * c1);
                  a0 = fmaf(a0, c0, __uint_as_float(v0[u]) * c1);
                  a1 = fmaf(a1, c0, __uint_as_float(v1[u]) * c1);
                }
              }
          }
          // What tells the producers to come back is what this workgroup stores in the coming phase, behind weights that this wave has requested since and
          // waited for.  A workgroup without a share of that phase, or a wave without a share of its K (rows of fewer than 1024), waits here.
          if (splits > 1 && (P.phase[BG_O].units < ncu || P.phase[BG_O].ksteps < BS_PASS)) vm_wait_all();
#pragma unroll
          for (int d = 0; d < HD; d += 64) {
            const int row = (g * G + hq) * HD + d + lane;
            bs_put(P, out + ((row >> 3) * slots + slot) * 8 + (row & 7), bs_split_word((d ? a1 : a0) / den));
          }
        });
        lds_barrier();
      }
      {                                                           // sequences that skip this layer: nothing of theirs is looked at, but the words must be there
        const unsigned bits = (unsigned)uni(kept[kl]) >> 16;
        const int lane = sk_lane_opaque(), nq = p.Hkv * G * HD;
        for (int j = 0; j < n; ++j)
          if (!((bits >> j) & 1))
            for (int row = (wg * (BS_THREADS / 64) + wave) * 64 + lane; row < nq; row += ncu * BS_THREADS) bs_put(P, out + ((row >> 3) * slots + j) * 8 + (row & 7), 0u);
      }
      if (uni(*bad)) return;
      if (streams) {
        cur = bs_seg(P, BG_O, layer_of(kl), pair);
        first_chunks(P.up_offset);
      } else {
        no_ring();
      }
    } else if (!streams) {
      no_ring();
    }
  }
}

}  // namespace first
