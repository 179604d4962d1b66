// The projections of the prompt pass on the matrix cores: C[M, N] = (Ah + Al)[M, K] . W[N, K]^T with activations split
// into two bf16 parts (see k_gemm_nt_bf16_split) and bf16 weights, fp32 accumulation.
//
// Both parts meet the same weight tile, so a K step costs 2 BM + BN rows of operands and 4 BM BN BK flops.  Operands go from
// global memory straight into LDS (buffer loads with an LDS destination, 16 bytes a lane; the descriptor covers the tile's
// rows, so rows past the end read as zeros and nothing is clamped).  A row's 16-byte chunks are permuted by its number - on the way
// in through the address each lane fetches - so that the 32 rows a wave reads at one K offset spread over all banks.
//
// What bounds it.  Long launches: the card's power - at 16384 rows the matrix cores are busy 60 % of the cycles of a clock that has
// dropped from 2.4 to 1.8 GHz, and the same launch on zeros is a quarter faster.  Up to there: LDS - a wave's 64 x 64 part of
// the tile reads 0.75 fragments of 1 KB an MFMA, and four SIMDs at full rate would read 96 and have 32 bytes a clock written for
// them of the 128 there are - so fragments of the next 16 columns of K are read while the present ones are multiplied, across
// the barrier between steps too, and gate / up takes 256 x 256 tiles (64 x 128 a wave: 0.5 fragments an MFMA) where
// they fill the chip.
//
// Measured alone, cold weights (matrix-core work, twice the useful flops; in brackets the same tiles with every fragment
// read behind its step's barrier, as they were): 1024 x 28672 x 4096 406 us = 1.19 PFLOP/s with 256 x 256 tiles (436 with 128 x 256),
// 16384 rows 5.96 ms = 1.29 (6.42); 1024 x 4096 x 14336 213 us = 1.13 with 128 x 256 tiles and two slices of K (234 with 64 x 256),
// 1024 x 6144 x 4096 94 us with 128 x 192 tiles (101 with 128 x 256); 826 x 5120 x 3072 58 us (70).  The library's plain bf16 product
// runs at 1.11 PFLOP/s on 1024 x 28672 x 4096, at 1.26 on 8192^3.
#pragma once
#include "step_kernel.h"

namespace first {

constexpr int PG_BK = 64;                       // K step that segments are counted in (a tile's own step: 64, or 32 where LDS is short)

// 16 bytes per lane from (descriptor base + voff + soff) to LDS byte lds_off + 16 * lane.  No vector register is written: nothing
// for the compiler to reuse too early; pg_wait / lds_barrier order it.  The LDS offset travels in m0, as an operand: it is the
// compiler that writes the register, so it knows (m0 written in the asm text would be a write it knows nothing of).
typedef int i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void pg_load_lds(uint32_t lds_off, uint32_t voff, i32x4_t rsrc, uint32_t soff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"{m0}"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
__device__ __forceinline__ i32x4_t pg_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  i32x4_t r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
template <int N> __device__ __forceinline__ void pg_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// place of a row's chunk: rows of 128 bytes (two rows are all banks), and of 64 bytes (four are)
__device__ __forceinline__ int pg_chunk(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }
template <int BK> __device__ __forceinline__ int pg_place(int row, int chunk) { return BK == 64 ? pg_chunk(row, chunk) : chunk ^ ((row >> 2) & 3); }

// One launch: up to three weight matrices applied to the same activations, their column tiles one after the other.
struct PgSeg { const bf16* W; float* C; int N; int tiles; };        // tiles = column tiles of this matrix
struct PgArgs {
  const bf16 *Ah, *Al;
  PgSeg seg[3];
  int nseg, M, K, accumulate;
  const bf16* Wu;               // gate/up launch: seg[0].W = gate, this = up, N = d_ffn
  bf16 *zh, *zl;                //   SiLU(gate) * up, split, [M, N]
  int gm, gn;                   // row tiles, column tiles of all matrices together
  int ks;                       // slices of K: 1, 2 or 4 (more than one with SPLIT and SEG = 4 only)
  float* part;                  // partial tiles of the slices, arrival counters per tile (zero between launches)
  unsigned* cnt;
};

// The order of additions does not depend on M, nor on the tile: a row of the result is the same bits whatever prompts share
// the launch.  With SEG = 4 (a property of the matrix, see pg_segments) K is four segments of whole steps of 64, each summed
// from zero, added in order; slices of K take whole segments, and the upper half's two travel apart.
//
// BM x BN tile, WGM x WGN waves, K steps of BK, S of them in the LDS ring.  S: three where they fit.  BK: 64, whole lines of the
// operands' rows; 32 for the 256 x 256 tile, whose steps of 64 would leave no room for a ring (and whose steps of 32 are as many
// products as the 128 x 256 tile's of 64).
// GU: the tile's BN weight rows are 32 (16 where a wave tile is 32 wide) gate rows and as many up rows in turn, so that
// a gate value and its up value sit in the same lane (in lanes 16 apart).
template <int BM, int BN, int WGM, int WGN, int BK, int S, bool GU, bool SPLIT, int SEG>
__global__ void __launch_bounds__(WGM * WGN * 64, 2) k_pgemm(PgArgs P) {
  constexpr int NW = WGM * WGN, TM = BM / WGM, TN = BN / WGN, IM = TM / 32, JN = TN / 32;
  constexpr int RB = BK * 2, RPL = 1024 / RB, CPR = BK / 8;      // bytes of a row, rows of a 1 KB load, chunks of a row
  constexpr int IA = BM / RPL / NW, IB = BN / RPL / NW;          // loads per wave and K step: each half of A; B
  constexpr int GI = JN >= 2 ? 32 : 16;                          // gate / up interleave
  static_assert(BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0 && TM % 32 == 0 && TN % 32 == 0, "tile shape");
  static_assert(SEG == 1 || (SEG == 4 && IM * JN <= 4), "segments of K: accumulators and their sum in registers");
  static_assert(!GU || JN == 1 || JN % 2 == 0, "a gate block and its up block in one wave");
  constexpr int STG = (2 * BM + BN) * RB;                        // LDS bytes of a K step
  constexpr int NKK = BK / 16, NL = 2 * IA + IB;
  extern __shared__ __align__(16) char pg_smem[];
  __shared__ int last_flag;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)pg_smem;
  const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
  const int K = P.K, M = P.M;

  // Workgroup -> tile.  Consecutive workgroups go to the eight XCDs in turn; each XCD gets a contiguous run of tiles, in
  // groups of eight row tiles (four of 256 rows) with the row tiles of a column next to each other: what runs on an XCD at a time is a
  // compact block of tiles whose operands its L2 holds (at 16384 x 28672 x 4096 column-major runs of all 128 row
  // tiles cost 5 to 50 %, depending on the tile).
  int id = blockIdx.x;
  {
    const int total = gridDim.x, per = total / 8, rem = total % 8, x = id % 8;
    id = x * per + min(x, rem) + id / 8;
  }
  const int slice = SPLIT ? id % P.ks : 0;
  if (SPLIT) id /= P.ks;
  const int tile = id;
  constexpr int GR = BM == 256 ? 4 : 8;
  const int grp = id / (GR * P.gn), in = id - grp * GR * P.gn, grn = min(GR, P.gm - grp * GR);
  const int m0 = (grp * GR + in % grn) * BM;
  int ct = in / grn, si = 0;
  if (!GU)
    while (si + 1 < P.nseg && ct >= P.seg[si].tiles) { ct -= P.seg[si].tiles; ++si; }
  const bf16* const W = P.seg[si].W;
  float* const C = P.seg[si].C;
  const int N = P.seg[si].N;
  const int n0 = ct * (GU ? BN / 2 : BN);
  const int rowsA = min(BM, M - m0), rowsB = min(GU ? BN / 2 : BN, N - n0);
  const i32x4_t rh = pg_rsrc(P.Ah + (size_t)m0 * K, (uint32_t)rowsA * K * 2);
  const i32x4_t rl = pg_rsrc(P.Al + (size_t)m0 * K, (uint32_t)rowsA * K * 2);
  const i32x4_t rb = pg_rsrc(W + (size_t)n0 * K, (uint32_t)rowsB * K * 2);
  const i32x4_t ru = GU ? pg_rsrc(P.Wu + (size_t)n0 * K, (uint32_t)rowsB * K * 2) : rb;

  // byte offset of this lane's chunk in each of the wave's loads; lane -> (row of the load, slot), slot holds chunk pg_place
  uint32_t va[IA], vb[IB];
  const int lrow = lane / CPR, lch = lane % CPR;
#pragma unroll
  for (int i = 0; i < IA; ++i) {
    const int r = (wave * IA + i) * RPL + lrow;
    va[i] = (uint32_t)r * K * 2 + pg_place<BK>(r, lch) * 16;
  }
#pragma unroll
  for (int i = 0; i < IB; ++i) {
    const int r = (wave * IB + i) * RPL + lrow;
    const int src = GU ? (r / (2 * GI)) * GI + r % GI : r;               // (a load's rows lie in one block of gate or of up rows)
    vb[i] = (uint32_t)src * K * 2 + pg_place<BK>(r, lch) * 16;
  }
  // segments of this workgroup and their steps
  const int n64 = (K + PG_BK - 1) / PG_BK, nsteps = (K + BK - 1) / BK;
  const int g0 = SPLIT ? SEG * slice / P.ks : 0, g1 = SPLIT && SEG > 1 ? SEG * (slice + 1) / P.ks : SEG;
  auto seg_start = [&](int g) { return min(n64 * g / SEG * (PG_BK / BK), nsteps); };
  const int s0 = seg_start(g0), s1 = seg_start(g1);
  const int tail_chunks = (K % BK) / 8;                                   // chunks of the last step that exist (0: all)
  auto issue = [&](int step, int slot) __attribute__((always_inline)) {
    // (uniform by construction; said again for the compiler, which does not see it through the loop: once a step, so that what a
    // load adds is a constant)
    const uint32_t b = (uint32_t)uni((int)(lds0 + (uint32_t)slot * STG)), so = (uint32_t)uni(step * RB);
    const uint32_t ba = b + (uint32_t)wave * IA * 1024, bb = b + 2 * BM * RB + (uint32_t)wave * IB * 1024;
    const bool cut = tail_chunks != 0 && step == nsteps - 1;
    auto off = [&](uint32_t v, int r) __attribute__((always_inline)) {   // past the row's end: out of the descriptor's range, reads as zeros
      return cut && pg_place<BK>(r, lch) >= tail_chunks ? 0x7ffffff0u : v;
    };
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const uint32_t v = off(va[i], (wave * IA + i) * RPL + lrow);
      pg_load_lds(ba + i * 1024, v, rh, so);
      pg_load_lds(ba + BM * RB + i * 1024, v, rl, so);
    }
#pragma unroll
    for (int i = 0; i < IB; ++i) {
      const int r8 = (wave * IB + i) * RPL;
      const bool up = GU && (r8 / GI) % 2 == 1;
      pg_load_lds(bb + i * 1024, off(vb[i], r8 + lrow), up ? ru : rb, so);
    }
  };
  floatx16_t acc[IM][JN], tot[SEG > 1 ? IM : 1][JN];
  auto zero = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  const int wm = (wave / WGN) * TM, wn = (wave % WGN) * TN;
  const int lr = lane & 31, lg = lane >> 5;
  // fragments of 16 columns of K: LDS offsets per lane, two sets of registers
  uint32_t oa[NKK], ob[NKK];
#pragma unroll
  for (int k = 0; k < NKK; ++k) {
    oa[k] = (wm + lr) * RB + pg_place<BK>(wm + lr, 2 * k + lg) * 16;
    ob[k] = 2 * BM * RB + (wn + lr) * RB + pg_place<BK>(wn + lr, 2 * k + lg) * 16;
  }
  bf16x8_t fa[2][2][IM], fb[2][JN];
  auto frags = [&](int buf, int slot, int k) __attribute__((always_inline)) {
    const char* base = pg_smem + slot * STG;
#pragma unroll
    for (int j = 0; j < JN; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8_t*>(base + ob[k] + j * 32 * RB);
#pragma unroll
    for (int i = 0; i < IM; ++i) fa[buf][1][i] = *reinterpret_cast<const bf16x8_t*>(base + oa[k] + BM * RB + i * 32 * RB);
#pragma unroll
    for (int i = 0; i < IM; ++i) fa[buf][0][i] = *reinterpret_cast<const bf16x8_t*>(base + oa[k] + i * 32 * RB);
  };
  auto mfma = [&](int buf) __attribute__((always_inline)) {
    // low halves before high halves; two products into the same accumulator are not back to back except where a wave has only one (32 x 128
    // tiles); with two row blocks a weight fragment's products follow each other (up to 4 % over products by row block: each fragment is needed later)
    if constexpr (IM > 1) {
#pragma unroll
      for (int j = 0; j < JN; ++j)
#pragma unroll
        for (int p = 1; p >= 0; --p)
#pragma unroll
          for (int i = 0; i < IM; ++i) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][p][i], fb[buf][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(8, 1, 0);
          }
      return;
    }
#pragma unroll
    for (int p = 1; p >= 0; --p)
#pragma unroll
      for (int i = 0; i < IM; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[buf][p][i], fb[buf][j], acc[i][j], 0, 0, 0);
  };
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (s0 + s < s1) issue(s0 + s, s);
  if (s0 + S - 1 < s1) pg_wait<NL * (S - 1)>(); else pg_wait<0>();
  lds_barrier();
  frags(0, 0, 0);
  zero();
  // the upper half of K on its own: its two segments are added to the lower half's sum one after the other
  const bool apart = SEG > 1 && SPLIT && P.ks == 2 && slice == 1;
  int slot = 0, s = s0;
  for (int sg = g0; sg < g1; ++sg) {
    for (const int e1 = seg_start(sg + 1); s < e1; ++s) {
      const int nslot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
      for (int k = 0; k < NKK; ++k) {
        if (k + 1 < NKK) {
          frags((k + 1) & 1, slot, k + 1);
        } else if (s + 1 < s1) {                 // every fragment of this step is read: its place in the ring is free once all waves say so
          if (s + S - 1 < s1) pg_wait<NL * (S - 2)>(); else pg_wait<0>();
          lds_barrier();
          if (s + S < s1) issue(s + S, slot);
          frags(0, nslot, 0);
        }
        mfma(k & 1);
      }
      slot = nslot;
    }
    if constexpr (SEG > 1) {                   // what the segments of this workgroup come to so far
      if (sg == g0) {
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int j = 0; j < JN; ++j) tot[i][j] = acc[i][j];
      } else if (!apart) {
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) tot[i][j][r] += acc[i][j][r];
      }
      if (sg + 1 < g1) zero();
    }
  }
  // Through a descriptor that ends with the tile's last row: rows past M (and, by an offset out of its range, columns past N)
  // read as zeros and are not written, without a branch per element.
  // D layout of the 32x32 MFMA: lane -> column (lane & 31); register r -> row 8 (r / 4) + 4 (lane / 32) + r % 4
  const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(uni(C + (size_t)m0 * N), (short)0, rowsA * N * 4, 0x00020000);
  // (a select per column, none per element: the compiler makes branches of those, with a wait for all loads in each)
  uint32_t colb[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) {
    const int col = n0 + wn + j * 32 + lr;
    colb[j] = (uint32_t)(wm + 4 * lg) * N * 4 + (col < N ? col * 4u : 0x40000000u);   // (a tile's rows are at most 2^30 bytes)
  }
  auto at = [&](int i, int j, int r) __attribute__((always_inline)) {
    uint32_t b = colb[j];
    asm volatile("" : "+v"(b));                // (formed where it is used: kept from a load to its store, the offsets take 64 registers)
    return (int)(b + (uint32_t)(i * 32 + 8 * (r >> 2) + (r & 3)) * N * 4);
  };
  if constexpr (SPLIT && SEG > 1) {
    // Slices of K (two or four): every workgroup stores its partial tile (accumulator order, 16 bytes a lane, write-through),
    // counts itself in, and the last one adds the slices as the segments are added - the sum does not depend on who is last.
    if (P.ks > 1) {
      constexpr size_t WF = (size_t)IM * JN * 1024;                      // floats of one wave's partial tile
      // (Stores the compiler knows, so that it sees that they read what the last MFMA is still writing, and without a scalar
      // offset: with one it takes the data registers for free at once, and overwriting them in the next instruction put
      // wrong values into one of the four words now and then.)
      auto put = [&](const floatx16_t (&from)[IM][JN], int slot) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(uni(P.part + (((size_t)tile * 4 + slot) * NW + wave) * WF), (short)0,
                                                                            (int)(WF * 4), 0x00020000);
#pragma unroll
        for (int i = 0; i < IM; ++i)
#pragma unroll
          for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const u32x4_t v = {__float_as_uint(from[i][j][4 * q]), __float_as_uint(from[i][j][4 * q + 1]),
                                 __float_as_uint(from[i][j][4 * q + 2]), __float_as_uint(from[i][j][4 * q + 3])};
              __builtin_amdgcn_raw_buffer_store_b128(v, rw, ((i * JN + j) * 4 + q) * 1024 + lane * 16, 0, 17);   // sc0 sc1
            }
      };
      put(tot, slice);
      if (apart) put(acc, 2);
      pg_wait<0>();
      __syncthreads();
      if (tid == 0) {
        const unsigned old = __hip_atomic_fetch_add(P.cnt + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = old == (unsigned)(P.ks - 1);
        if (last) __hip_atomic_store(P.cnt + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last_flag = last;
      }
      __syncthreads();
      if (!last_flag) return;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(uni(P.part + (size_t)tile * 4 * NW * WF), (short)0,
                                                                          (int)(4 * NW * WF * 4), 0x00020000);
      // blocks of 32 x 32, the next one (and what it is added to) on its way while one is added up: all of a 64 x 64 wave tile
      // at once would take every register there is
      floatx16_t p[2][4];
      float old[2][16];
      auto request = [&](int blk) __attribute__((always_inline)) {
        const int i = blk / JN, j = blk % JN, b = blk & 1;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q == 3 && P.ks == 2) continue;
          const int so = (int)(((size_t)q * NW + wave) * WF * 4);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const u32x4_t x = __builtin_amdgcn_raw_buffer_load_b128(rs, (blk * 4 + v) * 1024 + lane * 16, so, 17);   // sc0 sc1
#pragma unroll
            for (int e = 0; e < 4; ++e) p[b][q][4 * v + e] = __uint_as_float(x[e]);
          }
        }
        if (P.accumulate) {
#pragma unroll
          for (int r = 0; r < 16; ++r) old[b][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, at(i, j, r), 0, 0));
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) old[b][r] = 0.f;
        }
      };
      request(0);
#pragma unroll
      for (int blk = 0; blk < IM * JN; ++blk) {
        if (blk + 1 < IM * JN) request(blk + 1);
        const int b = blk & 1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float t = (p[b][0][r] + p[b][1][r]) + p[b][2][r];
          if (P.ks == 4) t += p[b][3][r];
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(old[b][r] + t), rc, at(blk / JN, blk % JN, r), 0, 0);
        }
      }
      return;
    }
  }
  if constexpr (SEG > 1) {
#pragma unroll
    for (int i = 0; i < IM; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = tot[i][j];
  }

  if constexpr (GU) {
    auto put = [&](int row, int col, float g, float u) __attribute__((always_inline)) {
      if (row >= M || col >= N) return;
      const float z = siluf(g) * u;
      const bf16 h = from_f32<bf16>(z);
      P.zh[(size_t)row * N + col] = h;
      P.zl[(size_t)row * N + col] = from_f32<bf16>(z - to_f32(h));
    };
#pragma unroll
    for (int i = 0; i < IM; ++i) {
      if constexpr (JN >= 2) {
#pragma unroll
        for (int j = 0; j < JN; j += 2)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            put(m0 + wm + i * 32 + 8 * (r >> 2) + 4 * lg + (r & 3), n0 + (wn + j * 32) / 2 + lr, acc[i][j][r], acc[i][j + 1][r]);
      } else {                                 // columns 0..15 gate, 16..31 up: each half finishes eight of the sixteen rows
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const bool hi = (lane & 16) != 0;
          const float give = hi ? acc[i][0][r] : acc[i][0][r + 1], keep = hi ? acc[i][0][r + 1] : acc[i][0][r];
          const float got = __shfl_xor(give, 16, 64);
          const int rr = hi ? r + 1 : r;
          put(m0 + wm + i * 32 + 8 * (rr >> 2) + 4 * lg + (rr & 3), n0 + wn / 2 + (lane & 15), hi ? got : keep, hi ? keep : got);
        }
      }
    }
  } else {
    // What is added to is requested as a whole (of a 64 x 128 wave tile: half by half) before any of it is used: a load, a wait and a
    // store per element were up to 64 memory round trips in a row, 50 to 80 us of the 4096 x 14336 projection of 1024 rows.
    constexpr int IG = IM * JN > 4 ? 1 : IM;
#pragma unroll
    for (int i0 = 0; i0 < IM; i0 += IG) {
      float old[IG][JN][16];
      if (P.accumulate) {
#pragma unroll
        for (int i = 0; i < IG; ++i)
#pragma unroll
          for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) old[i][j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, at(i0 + i, j, r), 0, 0));
      } else {
#pragma unroll
        for (int i = 0; i < IG; ++i)
#pragma unroll
          for (int j = 0; j < JN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) old[i][j][r] = 0.f;
      }
#pragma unroll
      for (int i = 0; i < IG; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(old[i][j][r] + acc[i0 + i][j][r]), rc, at(i0 + i, j, r), 0, 0);
    }
  }
}

}  // namespace first
