// bf16 GEMM on gfx950 matrix cores: C[M][N] = A[M][K] . B[N][K]^T with fp32
// accumulation and a fused epilogue per use in the verify forward pass:
//
//   EPI_QKV      q/k/v projections; rotary embedding of q and k; q goes to a
//                workspace buffer, k and v straight into the KV cache at the
//                node's slot S_b + node
//   EPI_RESID    o-projection / down-projection, added into the fp32
//                residual stream
//   EPI_GATE_UP  gate and up projections of the same features side by side,
//                emitting silu(gate) * up in bf16
//   EPI_ARGMAX   LM head: per row, the (max, lowest index) over each wave's
//                column slab, optionally also the fp32 logits
//
// Three kernels, chosen by pick_tile() and skinny_max_rows():
//   * many rows (over 128): 256 x 256 and 256 x 128 tiles whose two wave groups
//     run in opposite phases (see there);
//   * few rows: one work-group per 16 weight rows (see there);
//   * in between, the ring kernel: one work-group of 4 waves in a WM x WN grid,
//     output tile BM x BN (128 x 128 with 4 stages, 64 x 256 and 32 x 256 with
//     3, where the weights are streamed), each wave BM/WM x BN/WN built from
//     32 x 32 v_mfma_f32_32x32x16_bf16 blocks, K step 64:
//   * operand tiles move HBM/L2 -> LDS with global_load_lds_dwordx4 (no
//     register staging) into a ring of NS stages; the next NS-1 K steps are
//     in flight while the current one is multiplied, and one barrier per K
//     step both publishes the next stage and frees the oldest slot.  The
//     barrier waits only for this wave's LDS reads and for the loads of the
//     next stage (vmcnt counts the later stages out), never for the whole
//     ring.  A stage's wave-loads are issued in four parts between the MFMA
//     blocks, with their LDS destinations in scalar registers;
//   * each wave-load writes 1 KB = 8 tile rows of 128 bytes; the 16-byte chunk
//     index of row r is XOR-ed with (r >> 1) & 7, which makes the MFMA operand
//     reads (16 consecutive rows, one chunk) hit all 64 LDS banks once;
//   * fragments of the next 16-wide k-step are read from LDS into a second
//     register set while the current set feeds the MFMAs.
// Work-groups are dealt round-robin over the 8 XCDs; the tile order is remapped
// so that the M tiles sharing one weight tile run on one XCD and hit its L2.
//
// Products with too few output tiles to fill the CUs split K: each split
// writes its fp32 tile to a partial buffer and a second kernel sums the splits
// in a fixed order (bitwise reproducible) and applies the same epilogue.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace spec {

namespace {

constexpr size_t kPartialCap = 64ull << 20;   // bytes of split-K partials (workspace)

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ void load_lds16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (lds_void*)lds, 16, 0, 0);
}

// 16-byte chunk swizzle of tile row `row` (rows of 128 bytes): 16 consecutive
// rows reading one logical chunk hit 16 distinct 16-byte bank groups.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// Wait until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Work-group barrier for the LDS ring: this wave's LDS reads are complete
// (its slot may be refilled by any wave afterwards), but its direct-to-LDS
// loads of later stages stay in flight.  __syncthreads() would add a
// work-group fence, i.e. a wait for every outstanding global load, which
// would leave only one stage of lookahead however deep the ring.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Virtual-column mapping.  Column u of an output tile belongs to wave column
// wn = u / TN, MFMA block nb = (u % TN) / 32, lane column c = u % 32.  For
// EPI_QKV and EPI_GATE_UP, blocks (2p, 2p+1) of a wave column form pair
// P = (u % BN) / 64 of the tile: rotary partners (dims j, j + d/2) or
// (gate, up) of one feature.
template <int EPI, int BN>
__device__ __forceinline__ const bf16* weight_row(const GemmArgs& a, int tn, int u) {
  const int P = u >> 6, blk = (u >> 5) & 1, c = u & 31;
  if constexpr (EPI == EPI_QKV) {
    const int vs = tn * BN;
    const bf16* base;
    int local;
    if (vs < a.n0) { base = a.B0; local = vs; }
    else if (vs < a.n0 + a.n1) { base = a.B1; local = vs - a.n0; }
    else { base = a.B2; local = vs - a.n0 - a.n1; }
    const int hd = a.head_dim, qpd = hd / 64;
    const int head = P / qpd, dim = (P % qpd) * 32 + blk * (hd / 2) + c;
    return base + (size_t)(local + head * hd + dim) * a.K;
  } else if constexpr (EPI == EPI_GATE_UP) {
    const int f = tn * (BN / 2) + P * 32 + c;
    return (blk ? a.B1 : a.B0) + (size_t)f * a.K;
  } else {
    return a.B0 + (size_t)(tn * BN + u) * a.K;
  }
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Pair epilogues: (x1, x2) are the two members of pair P of tile tn, lane
// column c, output row `row`.
template <int BN>
__device__ __forceinline__ void epi_qkv(const GemmArgs& a, int row, int tn, int P, int c, float x1,
                                        float x2) {
  const int vs = tn * BN;
  int seg, local;
  if (vs < a.n0) { seg = 0; local = vs; }
  else if (vs < a.n0 + a.n1) { seg = 1; local = vs - a.n0; }
  else { seg = 2; local = vs - a.n0 - a.n1; }
  const int hd = a.head_dim, qpd = hd / 64, half = hd / 2;
  const int head = local / hd + P / qpd;
  const int fi = (P % qpd) * 32 + c;           // rotary frequency index = first dim of the pair
  if (seg < 2) {
    const float2 cs = a.rope_cs[(size_t)row * half + fi];
    const float y1 = x1 * cs.x - x2 * cs.y;
    const float y2 = x2 * cs.x + x1 * cs.y;
    x1 = y1;
    x2 = y2;
  }
  if (seg == 0) {
    bf16* pq = a.q_out + (size_t)row * a.n0 + head * hd + fi;
    pq[0] = (bf16)x1;
    pq[half] = (bf16)x2;
  } else {
    const TokInfo t = a.toks[row];
    const SampleInfo s = a.samples[t.sample];
    const int slot = s.seq_len + t.node;
    bf16* pk = a.kv_pool + s.kv_base +
               ((((size_t)a.layer * 2 + (seg - 1)) * a.n_kv_heads + head) * s.cap + slot) * hd + fi;
    pk[0] = (bf16)x1;
    pk[half] = (bf16)x2;
  }
}

template <int BN>
__device__ __forceinline__ void epi_gate_up(const GemmArgs& a, int row, int tn, int P, int c,
                                            float g, float u) {
  const int f = tn * (BN / 2) + P * 32 + c;
  a.act_out[(size_t)row * (a.N / 2) + f] = (bf16)(silu(g) * u);
}

// Work-group b runs on XCD b % 8, which receives q + 1 work-groups (x < r)
// or q (x >= r) for a grid of 8q + r.  Give each XCD a contiguous range of
// logical ids, so that the M tiles sharing a weight tile (adjacent ids)
// meet in one XCD's L2.
__device__ __forceinline__ int xcd_contiguous(int b, int total) {
  const int q = total >> 3, r = total & 7, x = b & 7, j = b >> 3;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
}

template <int EPI, int BM, int BN, int WM, int NS>
__global__ __launch_bounds__(256, 1) void gemm_ring_kernel(GemmArgs a) {
  constexpr int NW = 4, BK = 64, WN = NW / WM;
  constexpr int TM = BM / WM, TN = BN / WN, MB = TM / 32, NB = TN / 32;
  constexpr int ROWB = BK * 2, CPR = BK / 8, RPL = 1024 / ROWB;  // row bytes, chunks, rows per load
  constexpr int KS = BK / 16;                                     // MFMA k-steps per K step
  constexpr int A_BYTES = BM * ROWB, STAGE = (BM + BN) * ROWB;
  constexpr int A_LOADS = A_BYTES / 1024 / NW, B_LOADS = BN * ROWB / 1024 / NW;
  constexpr int LPW = A_LOADS + B_LOADS;    // wave-loads per wave and stage
  static_assert(MB >= 1 && NB >= 2 && A_LOADS >= 1 && B_LOADS >= 1, "tile shape");
  static_assert(A_BYTES % (1024 * NW) == 0 && BN * ROWB % (1024 * NW) == 0, "loads per wave");
  static_assert(NS >= 2 && (NS - 2) * LPW <= 63, "ring depth (vmcnt holds at most 63)");
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  // The wave index is made scalar so that every LDS destination (M0) of the
  // direct loads is computed in scalar registers.
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntm = (a.M + BM - 1) / BM;
  const int tiles = ntm * (a.N / BN);
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int tile = bid % tiles, split = bid / tiles;
  const int tm = tile % ntm, tn = tile / ntm;
  const int KT = a.K / BK / a.ksplit;            // K steps of this split
  const int k_off = split * KT * BK;

  // Wave-load j of this wave fills tile rows [(wave*LOADS + j)*RPL, +RPL);
  // lane l lands at row l/CPR, physical chunk l%CPR, so it fetches logical
  // chunk (l%CPR) ^ swz(row).
  const int lr = lane / CPR, lc = lane % CPR;
  const bf16* pa[A_LOADS];
  const bf16* pb[B_LOADS];
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int trow = (wave * A_LOADS + j) * RPL + lr;
    int row = tm * BM + trow;
    row = row < a.M ? row : a.M - 1;      // rows past M repeat the last row; never stored
    pa[j] = a.A + (size_t)row * a.K + k_off + ((lc ^ swz(trow)) << 3);
  }
#pragma unroll
  for (int j = 0; j < B_LOADS; ++j) {
    const int trow = (wave * B_LOADS + j) * RPL + lr;
    pb[j] = weight_row<EPI, BN>(a, tn, trow) + k_off + ((lc ^ swz(trow)) << 3);
  }
  // Part q of stage kt's loads (every KS-th wave-load), so that a stage's
  // loads are spread between the MFMA blocks of a K step instead of issued
  // in one burst.
  auto issue_q = [&](int kt, int slot, int q) {
    char* base = smem + slot * STAGE;
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j)
      if (j % KS == q) load_lds16(pa[j] + kt * BK, base + (wave * A_LOADS + j) * 1024);
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j)
      if (j % KS == q) load_lds16(pb[j] + kt * BK, base + A_BYTES + (wave * B_LOADS + j) * 1024);
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x16{};

  const int wm = wave / WN, wn = wave % WN;
  int arow[MB], brow[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) arow[i] = wm * TM + i * 32 + (lane & 31);
#pragma unroll
  for (int j = 0; j < NB; ++j) brow[j] = wn * TN + j * 32 + (lane & 31);

  bf16x8 fa[2][MB], fb[2][NB];
  auto load_frags = [&](const char* st, int ks, int set) {
    const int chunk = ks * 2 + (lane >> 5);
#pragma unroll
    for (int i = 0; i < MB; ++i)
      fa[set][i] = *(const bf16x8*)(st + arow[i] * ROWB + ((chunk ^ swz(arow[i])) << 4));
#pragma unroll
    for (int j = 0; j < NB; ++j)
      fb[set][j] = *(const bf16x8*)(st + A_BYTES + brow[j] * ROWB + ((chunk ^ swz(brow[j])) << 4));
  };
  auto mfmas = [&](int set) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
  };

  // Prologue: stages 0 .. NS-2 in flight, wait for stage 0.
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < KT) {
#pragma unroll
      for (int q = 0; q < KS; ++q) issue_q(st, st, q);
    }
  if (KT >= NS - 1) wait_vm<(NS - 2) * LPW>();
  else wait_vm<0>();
  ring_barrier();
  // Stage pk (slot ps) is issued part by part between the MFMA blocks of the
  // current step; -1 when none is left.
  int pk = NS - 1 < KT ? NS - 1 : -1, ps = NS - 1;
  if (pk >= 0) issue_q(pk, ps, 0);
  load_frags(smem, 0, 0);
  for (int kt = 0; kt < KT; ++kt) {
    const char* st = smem + (kt % NS) * STAGE;
#pragma unroll
    for (int ks = 0; ks + 1 < KS; ++ks) {
      load_frags(st, ks + 1, (ks + 1) & 1);
      if (pk >= 0) issue_q(pk, ps, ks + 1);
      mfmas(ks & 1);
    }
    pk = -1;
    if (kt + 1 < KT) {
      // Stage kt+1 has landed for every wave (stages kt+2 .. kt+NS-1 may
      // still be in flight), and every wave is done reading stage kt (its
      // last fragments are in registers): that slot takes stage kt+NS.
      if (kt + NS - 1 < KT) wait_vm<(NS - 2) * LPW>();
      else wait_vm<0>();
      ring_barrier();
      if (kt + NS < KT) {
        pk = kt + NS;
        ps = kt % NS;
        issue_q(pk, ps, 0);
      }
      load_frags(smem + ((kt + 1) % NS) * STAGE, 0, 0);
    }
    mfmas((KS - 1) & 1);
  }

  // Accumulator layout of a 32x32 block: lane l, element e holds
  // row 8*(e/4) + 4*(l/32) + e%4, column l%32.
  const int c = lane & 31;
  const int rbase = tm * BM + wm * TM + 4 * (lane >> 5);

  if (a.ksplit > 1) {
    // Raw fp32 tile of this split, virtual column order.
    float* out = a.partial + (size_t)split * a.M * a.N + tn * BN + wn * TN + c;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          if (row < a.M) out[(size_t)row * a.N + j * 32] = acc[i][j][e];
        }
    return;
  }

  if constexpr (EPI == EPI_RESID) {
    // Read a whole 32x32 block of the residual before writing any of it, so
    // the 16 loads per lane are in flight together.
    float* xcol = a.x + tn * BN + wn * TN + c;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        float xv[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          xv[e] = row < a.M ? xcol[(size_t)row * a.N + j * 32] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          if (row < a.M) xcol[(size_t)row * a.N + j * 32] = xv[e] + acc[i][j][e];
        }
      }
  } else if constexpr (EPI == EPI_GATE_UP) {
#pragma unroll
    for (int p = 0; p < NB / 2; ++p)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          if (row >= a.M) continue;
          epi_gate_up<BN>(a, row, tn, wn * (NB / 2) + p, c, acc[i][2 * p][e], acc[i][2 * p + 1][e]);
        }
  } else if constexpr (EPI == EPI_QKV) {
    // The same arithmetic as epi_qkv, with the segment and head taken once
    // per wave and, for each 32-row block, every row's rotary angles and
    // destination fetched before any is used, so those loads (and the
    // token -> sample -> cache slot chain of K and V rows) are in flight
    // together instead of one row after another.
    const int vs = tn * BN;
    const int seg = vs < a.n0 ? 0 : (vs < a.n0 + a.n1 ? 1 : 2);
    const int local = vs - (seg == 0 ? 0 : (seg == 1 ? a.n0 : a.n0 + a.n1));
    const int hd = a.head_dim, qpd = hd / 64, half = hd / 2;
#pragma unroll
    for (int p = 0; p < NB / 2; ++p) {
      const int P = wn * (NB / 2) + p;
      const int head = local / hd + P / qpd;
      const int fi = (P % qpd) * 32 + c;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        float2 cs[16];
        bf16* dst[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          row = row < a.M ? row : a.M - 1;        // loads only; stores are guarded below
          cs[e] = seg < 2 ? a.rope_cs[(size_t)row * half + fi] : float2{1.f, 0.f};
        }
        if (seg == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
            dst[e] = a.q_out + (size_t)row * a.n0 + head * hd + fi;
          }
        } else {
          int smp[16], node[16];
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
            row = row < a.M ? row : a.M - 1;
            smp[e] = a.toks[row].sample;
            node[e] = a.toks[row].node;
          }
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const SampleInfo sv = a.samples[smp[e]];
            dst[e] = a.kv_pool + sv.kv_base +
                     ((((size_t)a.layer * 2 + (seg - 1)) * a.n_kv_heads + head) * sv.cap + sv.seq_len +
                      node[e]) * hd + fi;
          }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
          if (row >= a.M) continue;
          float x1 = acc[i][2 * p][e], x2 = acc[i][2 * p + 1][e];
          if (seg < 2) {
            const float y1 = x1 * cs[e].x - x2 * cs[e].y;
            const float y2 = x2 * cs[e].x + x1 * cs[e].y;
            x1 = y1;
            x2 = y2;
          }
          dst[e][0] = (bf16)x1;
          dst[e][half] = (bf16)x2;
        }
      }
    }
  } else {  // EPI_ARGMAX: one partial (max, lowest index) per row and wave slab of TN columns
    const int col0 = tn * BN + wn * TN + c;
    const int parts = a.N / TN;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = rbase + i * 32 + 8 * (e >> 2) + (e & 3);
        float v = acc[i][0][e];
        int idx = col0;
#pragma unroll
        for (int j = 1; j < NB; ++j)
          if (acc[i][j][e] > v) { v = acc[i][j][e]; idx = col0 + 32 * j; }
        if (a.logits != nullptr && row < a.M) {
#pragma unroll
          for (int j = 0; j < NB; ++j) a.logits[(size_t)row * a.N + col0 + 32 * j] = acc[i][j][e];
        }
#pragma unroll
        for (int m = 16; m >= 1; m >>= 1) {
          const float ov = __shfl_xor(v, m);
          const int oi = __shfl_xor(idx, m);
          if (ov > v || (ov == v && oi < idx)) { v = ov; idx = oi; }
        }
        if (c == 0 && row < a.M) {
          a.part_val[(size_t)row * parts + tn * WN + wn] = v;
          a.part_idx[(size_t)row * parts + tn * WN + wn] = idx;
        }
      }
  }
}

// ---- many rows: 256-row tiles, two wave groups in opposite phases ---------
//
// Both kernels below run 8 waves, two per SIMD, as two groups of four (group g
// = wave / 4; waves w and w + 4 share a SIMD).  A K step is cut into phases,
// each a memory part (fragment reads from LDS, direct loads of a later K step)
// and an MFMA part, separated by work-group barriers; group 1 runs one barrier
// behind group 0, so on every SIMD one wave's MFMAs always meet the other
// wave's memory part and the matrix core does not wait for LDS.  (In the ring
// kernel above all waves read, then all multiply.)  Measured on the gate/up
// product of the 8B shape (28672 x 4096, weights from HBM), us at 512 / 1024 /
// 4096 rows: ring kernel 150 / 253 / 878, these phases with the same 32x32x16
// instructions 124 / 232 / 768.  The loop then issues MFMAs in 97 % of its
// cycles and the card's power limit sets the clock (about 1.4 GHz), so energy
// per product counts: 16x16x32 instructions, whose accumulator traffic per flop
// is half, sustain 2.06 against 1.83 PFLOP/s in a loop of MFMAs alone, and take
// the same product to 106 / 213 / 699 us (1.38 PFLOP/s at 4096 rows).
//
// The products are taken as D = W . A^T, so a lane's four accumulators of a
// 16 x 16 block are four consecutive output columns of one row: acc[i][j][e] =
// row 16 i + lane % 16, column 16 j + 4 (lane / 16) + e of the wave's tile.
// Every output goes out as 8 or 16 bytes per lane.

typedef __attribute__((address_space(3))) char lds_char;

// Direct global -> LDS load of 16 bytes per lane from base + voff to the
// wave-uniform LDS address `lds` + 16 * lane.  In assembly, so that the
// compiler does not wait for it at the next LDS read; the kernels' own vmcnt
// waits and barriers order it.
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
               : "memory", "m0");
}

// Barrier that no instruction is scheduled across.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Output tile of logical work-group id `tile`.  Up to 8 M tiles: all M tiles
// of a weight tile in a row.  More: blocks of 8 weight tiles x 4 M tiles, the
// 32 tiles an XCD runs at a time, so that its L2 is filled with 12 operand
// tiles instead of 2 + ntm (gate/up at 8192 rows 1424 -> 1274 us, at 4096 rows
// 684 -> 677 us, at 2048 rows 379 -> 387 us: hence the line).
__device__ __forceinline__ void tile_at(int tile, int ntm, int ntn, int* tm, int* tn) {
  constexpr int GN = 8, GM = 4;
  if (ntm <= 8) {
    *tm = tile % ntm;
    *tn = tile / ntm;
    return;
  }
  const int gi = tile / (GN * ntm), rem = tile % (GN * ntm);
  const int cols = min(GN, ntn - gi * GN), panel = rem / (GM * cols), in = rem - panel * GM * cols;
  const int rows = min(GM, ntm - panel * GM);
  *tm = panel * GM + in % rows;
  *tn = gi * GN + in / rows;
}

// The epilogues.  The wave's tile starts at row row0 and column col0 (a
// multiple of 64) of tile (tm, tn); columns j = 0, 1 (mod 4) and their partners
// j + 2 form the pairs of weight_row().
template <int EPI, int BM, int BN, int MB, int NB>
__device__ __forceinline__ void epilogue_rows(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tm, int tn,
                                              int row0, int col0, int split, int lane) {
  const int m = tm * BM + row0 + (lane & 15), c4 = 4 * (lane >> 4);
  if (a.ksplit > 1) {      // raw fp32 tile of this split, virtual column order
    float* out = a.partial + (size_t)split * a.M * a.N + tn * BN + col0 + c4;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = m + 16 * i;
      if (row < a.M)
#pragma unroll
        for (int j = 0; j < NB; ++j) *(f32x4*)(out + (size_t)row * a.N + 16 * j) = acc[i][j];
    }
    return;
  }
  if constexpr (EPI == EPI_RESID) {
    float* x = a.x + tn * BN + col0 + c4;
#pragma unroll
    for (int i0 = 0; i0 < MB; i0 += 2) {     // two rows' residuals in flight together
      f32x4 xv[2][NB];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = m + 16 * (i0 + i);
        if (row < a.M)
#pragma unroll
          for (int j = 0; j < NB; ++j) xv[i][j] = *(const f32x4*)(x + (size_t)row * a.N + 16 * j);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = m + 16 * (i0 + i);
        if (row < a.M)
#pragma unroll
          for (int j = 0; j < NB; ++j) *(f32x4*)(x + (size_t)row * a.N + 16 * j) = xv[i][j] + acc[i0 + i][j];
      }
    }
  } else if constexpr (EPI == EPI_GATE_UP) {
    bf16* out = a.act_out + tn * (BN / 2) + col0 / 2 + c4;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = m + 16 * i;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (j & 2) continue;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (bf16)(silu(acc[i][j][e]) * acc[i][j + 2][e]);
        if (row < a.M) *(bf16x4*)(out + (size_t)row * (a.N / 2) + (j >> 2) * 32 + (j & 1) * 16) = v;
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    static_assert(NB == 4, "one pair of 32-column blocks per wave");
    const int vs = tn * BN;
    const int seg = vs < a.n0 ? 0 : (vs < a.n0 + a.n1 ? 1 : 2);
    const int local = vs - (seg == 0 ? 0 : (seg == 1 ? a.n0 : a.n0 + a.n1));
    const int hd = a.head_dim, qpd = hd / 64, half = hd / 2, P = col0 >> 6;
    const int head = local / hd + P / qpd, fi = (P % qpd) * 32 + c4;
    // Every row's destination first (for K and V through token -> sample ->
    // cache slot), so that those dependent loads are in flight together.
    bf16* dst[MB];
    if (seg == 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i) dst[i] = a.q_out + (size_t)(m + 16 * i) * a.n0 + head * hd + fi;
    } else {
      int smp[MB], node[MB];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int row = min(m + 16 * i, a.M - 1);
        smp[i] = a.toks[row].sample;
        node[i] = a.toks[row].node;
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const SampleInfo sv = a.samples[smp[i]];
        dst[i] = a.kv_pool + sv.kv_base +
                 ((((size_t)a.layer * 2 + (seg - 1)) * a.n_kv_heads + head) * sv.cap + sv.seq_len +
                  node[i]) * hd + fi;
      }
    }
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = m + 16 * i;
      if (row >= a.M) continue;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f32x4 x1 = acc[i][j], x2 = acc[i][j + 2];
        if (seg < 2) {
          const float* cs = (const float*)(a.rope_cs + (size_t)row * half + fi + 16 * j);
          const f32x4 t0 = *(const f32x4*)cs, t1 = *(const f32x4*)(cs + 4);   // (cos, sin) x 4
          const float co[4] = {t0[0], t0[2], t1[0], t1[2]}, si[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float y1 = x1[e] * co[e] - x2[e] * si[e];
            const float y2 = x2[e] * co[e] + x1[e] * si[e];
            x1[e] = y1;
            x2[e] = y2;
          }
        }
        bf16x4 v1, v2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v1[e] = (bf16)x1[e];
          v2[e] = (bf16)x2[e];
        }
        *(bf16x4*)(dst[i] + 16 * j) = v1;
        *(bf16x4*)(dst[i] + 16 * j + half) = v2;
      }
    }
  } else {  // EPI_ARGMAX: one partial (max, lowest index) per row and wave slab of 16 NB columns
    const int colb = tn * BN + col0 + c4, parts = a.N / (16 * NB);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int row = m + 16 * i;
      float v = -INFINITY;
      int idx = 0x7fffffff;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (acc[i][j][e] > v) { v = acc[i][j][e]; idx = colb + 16 * j + e; }
      if (a.logits != nullptr && row < a.M) {
#pragma unroll
        for (int j = 0; j < NB; ++j) *(f32x4*)(a.logits + (size_t)row * a.N + colb + 16 * j) = acc[i][j];
      }
#pragma unroll
      for (int x = 32; x >= 16; x >>= 1) {
        const float ov = __shfl_xor(v, x);
        const int oi = __shfl_xor(idx, x);
        if (ov > v || (ov == v && oi < idx)) { v = ov; idx = oi; }
      }
      if (lane < 16 && row < a.M) {
        const size_t at = (size_t)row * parts + (tn * BN + col0) / (16 * NB);
        a.part_val[at] = v;
        a.part_idx[at] = idx;
      }
    }
  }
}

// 256 x 256 tiles, 64-wide K steps in two stages of 64 KB.  Group g holds rows
// 128 g .., wave q = wave % 4 of it columns 64 q ..: 128 x 64 per wave.  Every
// step is four phases of 16 MFMAs, one quadrant (64 rows x 32 columns, K = 64)
// each: (A0, B0), (A0, B1), (A1, B1), (A1, B0), A0 / A1 the halves of the
// wave's rows and B0 / B1 of its columns.  A half is read into registers once,
// B0 of the next step in the last phase, so the LDS rows of a half are free one
// phase after their read and take the step after next: phases 0 .. 3 load A1
// (next step), B0, A0, B1 (step after next), two wave-loads per wave each, and
// every load has five phases (2.1 of 2.6 thousand cycles) to arrive.
template <int EPI>
__global__ __launch_bounds__(512, 2) void gemm_256x256_kernel(GemmArgs a) {
  constexpr int BM = 256, BN = 256, ROWB = 128, STAGE = (BM + BN) * ROWB, BOFF = BM * ROWB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = wave >> 2, wn = wave & 3;
  const int ntm = (a.M + BM - 1) / BM, ntn = a.N / BN, tiles = ntm * ntn;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int split = bid / tiles;
  int tm, tn;
  tile_at(bid % tiles, ntm, ntn, &tm, &tn);
  const int KT = a.K / 64 / a.ksplit;            // K steps of this split (even)
  const size_t k_off = (size_t)split * KT * 64;

  // Wave-load j of half hh: 8 tile rows of 128 bytes; lane l lands at row l / 8,
  // chunk l % 8, so it fetches logical chunk (l % 8) ^ swz(row).
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t va[2][2], vb[2][2], la[2][2], lb[2][2];
  const int mlast = a.M - 1 - tm * BM;           // rows past M repeat the last row; never stored
  const bf16* abase = a.A + (size_t)tm * BM * a.K + k_off;
  const bf16* bbase[2] = {weight_row<EPI, BN>(a, tn, 0) + k_off, weight_row<EPI, BN>(a, tn, 32) + k_off};
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = wave * 2 + j;
      const int ra = (c >> 3) * 128 + hh * 64 + (c & 7) * 8, rb = (c >> 2) * 64 + hh * 32 + (c & 3) * 8;
      va[hh][j] = (uint32_t)min(ra + lr, mlast) * a.K * 2 + ((lc ^ swz(ra + lr)) << 4);
      vb[hh][j] = (uint32_t)((const char*)(weight_row<EPI, BN>(a, tn, rb + lr) + k_off) - (const char*)bbase[hh]) +
                  ((lc ^ swz(rb + lr)) << 4);
      la[hh][j] = ra * ROWB;
      lb[hh][j] = BOFF + rb * ROWB;
    }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
  auto load_a = [&](int kt, int buf, int hh) {
    const char* src = (const char*)abase + (size_t)kt * ROWB;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(src, va[hh][j], lds0 + buf * STAGE + la[hh][j]);
  };
  auto load_b = [&](int kt, int buf, int hh) {
    const char* src = (const char*)bbase[hh] + (size_t)kt * ROWB;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(src, vb[hh][j], lds0 + buf * STAGE + lb[hh][j]);
  };

  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};
  // Fragments [16-row block][K half]; B0 of the even and odd steps apart, as
  // the next step's is read while this step's is in use.
  bf16x8 fa[4][2], fb0[2][2][2], fb1[2][2];
  const int r = lane & 15;
  uint32_t ro[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) ro[ks] = r * ROWB + (((4 * ks + (lane >> 4)) ^ swz(r)) << 4);
  const char* arows = smem + g * 128 * ROWB;
  const char* brows = smem + BOFF + wn * 64 * ROWB;
  auto read_a = [&](int buf, int hh) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        fa[i][ks] = *(const bf16x8*)(arows + buf * STAGE + (hh * 64 + i * 16) * ROWB + ro[ks]);
  };
  auto read_b = [&](int buf, int hh, bf16x8 (&f)[2][2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        f[j][ks] = *(const bf16x8*)(brows + buf * STAGE + (hh * 32 + j * 16) * ROWB + ro[ks]);
  };
  auto quadrant = [&](int ih, int jh, bf16x8 (&f)[2][2]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[ih * 4 + i][jh * 2 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              f[j][ks], fa[i][ks], acc[ih * 4 + i][jh * 2 + j], 0, 0, 0);
  };
  // End of a phase's memory part: the loads that the next phase's reads need
  // (those issued five phases ago; `w` newer ones of this wave may be in
  // flight) have landed, and after the barrier every wave's have.
  auto multiply = [&](auto w, int ih, int jh, bf16x8 (&f)[2][2]) {
    wait_vm<decltype(w)::value>();
    phase_barrier();
    wait_lds();
    quadrant(ih, jh, f);
    phase_barrier();
  };
  // One K step in stage `buf`.  LEFT: steps after this one (2 = two or more).
  auto kstep = [&](int kt, auto buf_, auto left_) {
    constexpr int buf = decltype(buf_)::value, LEFT = decltype(left_)::value;
    constexpr int W0 = LEFT == 0 ? 2 : 10, W1 = LEFT == 2 ? 10 : LEFT == 1 ? 8 : 0,
                  W2 = LEFT == 2 ? 10 : LEFT == 1 ? 6 : 0, W3 = LEFT == 2 ? 10 : LEFT == 1 ? 4 : 0;
    read_a(buf, 0);
    if constexpr (LEFT >= 1) load_a(kt + 1, buf ^ 1, 1);
    multiply(std::integral_constant<int, W0>{}, 0, 0, fb0[buf]);
    read_b(buf, 1, fb1);
    if constexpr (LEFT == 2) load_b(kt + 2, buf, 0);
    multiply(std::integral_constant<int, W1>{}, 0, 1, fb1);
    read_a(buf, 1);
    if constexpr (LEFT == 2) load_a(kt + 2, buf, 0);
    multiply(std::integral_constant<int, W2>{}, 1, 1, fb1);
    if constexpr (LEFT >= 1) read_b(buf ^ 1, 0, fb0[buf ^ 1]);
    if constexpr (LEFT == 2) load_b(kt + 2, buf, 1);
    multiply(std::integral_constant<int, W3>{}, 1, 0, fb0[buf]);
  };

  load_b(0, 0, 0);
  load_a(0, 0, 0);
  load_b(0, 0, 1);
  load_a(0, 0, 1);
  load_b(1, 1, 0);
  load_a(1, 1, 0);
  load_b(1, 1, 1);
  wait_vm<10>();                                 // B0 and A0 of step 0
  phase_barrier();
  if (g == 1) phase_barrier();                   // group 1 runs one barrier behind
  read_b(0, 0, fb0[0]);
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  for (int kt = 0; kt < KT - 2; kt += 2) {
    kstep(kt, I0{}, I2{});
    kstep(kt + 1, I1{}, I2{});
  }
  kstep(KT - 2, I0{}, I1{});
  kstep(KT - 1, I1{}, I0{});
  if (g == 0) phase_barrier();
  epilogue_rows<EPI, BM, BN, 8, 4>(a, acc, tm, tn, g * 128, wn * 64, split, lane);
}

// 256 x 128 tiles, 64-wide K steps in three stages of 48 KB, for products that
// 256 x 256 tiles leave CUs idle on.  Waves in a 4 x 2 grid of 64 x 64 (group g
// = rows 128 g ..); two phases of 16 MFMAs per step, K = 32 each.  Stage kt + 2
// is loaded during step kt, into the stage that step kt - 1 has finished with.
template <int EPI>
__global__ __launch_bounds__(512, 2) void gemm_256x128_kernel(GemmArgs a) {
  constexpr int BM = 256, BN = 128, ROWB = 128, STAGE = (BM + BN) * ROWB, BOFF = BM * ROWB;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = wave >> 2, wm = wave >> 1, wn = wave & 1;
  const int ntm = (a.M + BM - 1) / BM, ntn = a.N / BN, tiles = ntm * ntn;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int split = bid / tiles;
  int tm, tn;
  tile_at(bid % tiles, ntm, ntn, &tm, &tn);
  const int KT = a.K / 64 / a.ksplit;            // at least 2
  const size_t k_off = (size_t)split * KT * 64;

  // Wave-loads as above: wave w loads A rows 32 w .. and weight rows 16 w ..
  // (which lie in one 32-row block, of one weight matrix).
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t va[4], vb[2];
  const int mlast = a.M - 1 - tm * BM;
  const bf16* abase = a.A + (size_t)tm * BM * a.K + k_off;
  const bf16* bbase = weight_row<EPI, BN>(a, tn, (wave >> 1) * 32) + k_off;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ra = (wave * 4 + j) * 8 + lr;
    va[j] = (uint32_t)min(ra, mlast) * a.K * 2 + ((lc ^ swz(ra)) << 4);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int rb = (wave * 2 + j) * 8 + lr;
    vb[j] = (uint32_t)((const char*)(weight_row<EPI, BN>(a, tn, rb) + k_off) - (const char*)bbase) +
            ((lc ^ swz(rb)) << 4);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
  const uint32_t lds_a = lds0 + wave * 32 * ROWB, lds_b = lds0 + BOFF + wave * 16 * ROWB;
  auto load_first = [&](int kt, uint32_t st) {
    const char* src = (const char*)abase + (size_t)kt * ROWB;
#pragma unroll
    for (int j = 0; j < 3; ++j) dma16(src, va[j], lds_a + st + j * 1024);
  };
  auto load_rest = [&](int kt, uint32_t st) {
    dma16((const char*)abase + (size_t)kt * ROWB, va[3], lds_a + st + 3072);
    const char* src = (const char*)bbase + (size_t)kt * ROWB;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16(src, vb[j], lds_b + st + j * 1024);
  };

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};
  bf16x8 fa[4], fb[4];
  const int r = lane & 15;
  uint32_t ro[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) ro[ks] = r * ROWB + (((4 * ks + (lane >> 4)) ^ swz(r)) << 4);
  const char* arows = smem + wm * 64 * ROWB;
  const char* brows = smem + BOFF + wn * 64 * ROWB;
  auto read_frags = [&](uint32_t st, int ks) {
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = *(const bf16x8*)(arows + st + i * 16 * ROWB + ro[ks]);
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[j] = *(const bf16x8*)(brows + st + j * 16 * ROWB + ro[ks]);
  };
  auto multiply = [&]() {
    phase_barrier();
    wait_lds();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    phase_barrier();
  };

  load_first(0, 0);
  load_rest(0, 0);
  load_first(1, STAGE);
  load_rest(1, STAGE);
  wait_vm<6>();                                  // stage 0
  phase_barrier();
  if (g == 1) phase_barrier();                   // group 1 runs one barrier behind
  uint32_t st = 0, fill = 2 * STAGE;             // stage being read, stage being filled
  for (int kt = 0; kt < KT; ++kt) {
    const bool more = kt + 2 < KT;
    read_frags(st, 0);
    if (more) load_first(kt + 2, fill);
    multiply();
    read_frags(st, 1);
    if (more) {
      load_rest(kt + 2, fill);
      wait_vm<6>();                              // stage kt + 1 has landed
    } else {
      wait_vm<0>();
    }
    multiply();
    st = st == 2 * STAGE ? 0 : st + STAGE;
    fill = fill == 2 * STAGE ? 0 : fill + STAGE;
  }
  if (g == 0) phase_barrier();
  epilogue_rows<EPI, BM, BN, 4, 4>(a, acc, tm, tn, wm * 64, wn * 64, split, lane);
}

// ---- few rows: the product is a stream of the weight rows -----------------
//
// One work-group of 4 waves owns one unit of 16 weight rows and splits K into
// four quarters, one per wave.  A wave multiplies with
// v_mfma_f32_16x16x32_bf16: A = the activation rows (zero from row M on),
// B = its 16 weight rows; lane l loads 16 bytes of row l % 16 at k-offset
// 8 (l / 16), so a wave reads 512 contiguous bytes of each row per 256-wide
// step, and the next step's loads are in flight while the current one is
// multiplied.  The quarters' 16 x 16 tiles meet in LDS and wave 0 sums them
// in wave order (a fixed order: bitwise reproducible) and applies the
// epilogue; no K split leaves the work-group, so no reduction kernel follows
// (a residual product leaves its RMSNorm to the caller).  Units: QKV = 8
// rotary pairs (dims j, j + d/2) of one head, GATE_UP = 8 (gate, up)
// features, RESID = 16 output columns.  Every unit reads all M activation
// rows, so the activation bytes grow with M against a fixed weight stream;
// past skinny_max_rows() the tile kernel's 256-row weight tiles win, and the
// LM head always takes the tile kernel.  Accumulator layout of the 16 x 16
// block: lane l, element i holds activation row 4 (l / 16) + i and unit row
// l % 16.
constexpr int kSkinnyRows = 16;
// Rows up to which a product takes this path (measured on the 8B shape
// against the tile kernel with its K splits): q/k/v and gate/up up to 4 rows
// (at 8 rows the activation re-reads already cost more than the saved
// reductions); the residual products up to 8 (at 16 rows the RMSNorm that
// then runs on its own costs more than the fused split-K reduction it
// replaces).
template <int EPI>
constexpr int skinny_max_rows() { return EPI == EPI_RESID ? 8 : 4; }

template <int EPI>
__device__ __forceinline__ const bf16* skinny_row(const GemmArgs& a, int unit, int c) {
  if constexpr (EPI == EPI_QKV) {
    const int hd = a.head_dim, upd = hd / 16;       // units per head
    const int head_all = unit / upd, jb = unit % upd;
    const int nh0 = a.n0 / hd, nh1 = a.n1 / hd;
    const bf16* base;
    int head;
    if (head_all < nh0) { base = a.B0; head = head_all; }
    else if (head_all < nh0 + nh1) { base = a.B1; head = head_all - nh0; }
    else { base = a.B2; head = head_all - nh0 - nh1; }
    const int dim = c < 8 ? jb * 8 + c : hd / 2 + jb * 8 + (c - 8);
    return base + (size_t)(head * hd + dim) * a.K;
  } else if constexpr (EPI == EPI_GATE_UP) {
    const int f = unit * 8 + (c & 7);
    return (c < 8 ? a.B0 : a.B1) + (size_t)f * a.K;
  } else {
    return a.B0 + (size_t)(unit * kSkinnyRows + c) * a.K;
  }
}

template <int EPI>
__global__ __launch_bounds__(256) void skinny_gemm_kernel(GemmArgs a) {
  static_assert(EPI != EPI_ARGMAX, "the LM head streams its rows through the tile kernel");
  __shared__ f32x4 red[4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, kq = lane >> 4;
  const int unit = blockIdx.x;
  const int kw = a.K / 4;                            // K of this wave (a multiple of 32)
  const int k0 = wave * kw, k1 = k0 + kw;
  const bf16* wrow = skinny_row<EPI>(a, unit, c) + kq * 8;
  const bool arow_ok = c < a.M;
  const bf16* arow = a.A + (size_t)(arow_ok ? c : 0) * a.K + kq * 8;

  constexpr int KB = 8;                              // 32-wide k-blocks per step
  bf16x8 bw[2][KB], ba[2][KB];
  auto load = [&](int set, int k) {
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      const int kk = k + j * 32;
      const bool in = kk < k1;
      bw[set][j] = in ? *(const bf16x8*)(wrow + kk) : bf16x8{};
      ba[set][j] = in && arow_ok ? *(const bf16x8*)(arow + kk) : bf16x8{};
    }
  };
  f32x4 acc = f32x4{};
  auto mfmas = [&](int set) {
#pragma unroll
    for (int j = 0; j < KB; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ba[set][j], bw[set][j], acc, 0, 0, 0);
  };
  load(0, k0);
  for (int k = k0; k < k1; k += 2 * KB * 32) {
    if (k + KB * 32 < k1) load(1, k + KB * 32);
    mfmas(0);
    if (k + KB * 32 >= k1) break;
    if (k + 2 * KB * 32 < k1) load(0, k + 2 * KB * 32);
    mfmas(1);
  }

  const int m0 = 4 * kq;                             // first activation row of this lane's elements
  {
    red[wave][lane] = acc;
    __syncthreads();
    if (wave != 0) return;
    f32x4 t = red[0][lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) t += red[w][lane];
    if constexpr (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + i;
        if (m < a.M) a.x[(size_t)m * a.N + unit * kSkinnyRows + c] += t[i];
      }
    } else if constexpr (EPI == EPI_GATE_UP) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float u = __shfl_xor(t[i], 8);         // lanes c and c + 8: gate and up of one feature
        const int m = m0 + i;
        if (c < 8 && m < a.M) a.act_out[(size_t)m * (a.N / 2) + unit * 8 + c] = (bf16)(silu(t[i]) * u);
      }
    } else {  // EPI_QKV: lanes c < 8 hold dims j, lanes c + 8 their partners j + d/2
      const int hd = a.head_dim, half = hd / 2, upd = hd / 16;
      const int head_all = unit / upd, jb = unit % upd;
      const int nh0 = a.n0 / hd, nh1 = a.n1 / hd;
      const int seg = head_all < nh0 ? 0 : (head_all < nh0 + nh1 ? 1 : 2);
      const int head = head_all - (seg == 0 ? 0 : (seg == 1 ? nh0 : nh0 + nh1));
      const int j = jb * 8 + (c & 7);               // rotary frequency index of the pair
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float other = __shfl_xor(t[i], 8);
        const int m = m0 + i;
        if (m >= a.M) continue;
        const float x1 = c < 8 ? t[i] : other, x2 = c < 8 ? other : t[i];
        float y = t[i];
        if (seg < 2) {
          const float2 cs = a.rope_cs[(size_t)m * half + j];
          y = c < 8 ? x1 * cs.x - x2 * cs.y : x2 * cs.x + x1 * cs.y;
        }
        const int dim = c < 8 ? j : j + half;
        if (seg == 0) {
          a.q_out[(size_t)m * a.n0 + head * hd + dim] = (bf16)y;
        } else {
          const TokInfo tk = a.toks[m];
          const SampleInfo sv = a.samples[tk.sample];
          a.kv_pool[sv.kv_base + ((((size_t)a.layer * 2 + (seg - 1)) * a.n_kv_heads + head) * sv.cap +
                                  sv.seq_len + tk.node) * hd + dim] = (bf16)y;
        }
      }
    }
  }
}

template <int EPI>
hipError_t launch_skinny(const GemmArgs& a, hipStream_t s) {
  long grid;
  if constexpr (EPI == EPI_QKV) grid = (long)(a.n0 + a.n1 + a.n2) / kSkinnyRows;
  else grid = (long)a.N / kSkinnyRows;
  if (a.norm_done) *a.norm_done = false;
  skinny_gemm_kernel<EPI><<<(unsigned)grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

// Sum the K splits in split order and apply the epilogue.  Thread (row,
// group g of 64 virtual columns, lane column c) owns virtual columns g*64 + c
// and g*64 + 32 + c: pair (g % (BN/64)) of tile g / (BN/64), or two residual
// columns.
template <int EPI, int BN>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int half_n = a.N / 2;
  if (idx >= (size_t)a.M * half_n) return;
  const int row = (int)(idx / half_n), rem = (int)(idx % half_n);
  const int g = rem >> 5, c = rem & 31;
  const size_t base = (size_t)row * a.N + g * 64 + c;
  float x1 = 0.f, x2 = 0.f;
  for (int s = 0; s < a.ksplit; ++s) {
    x1 += a.partial[(size_t)s * a.M * a.N + base];
    x2 += a.partial[(size_t)s * a.M * a.N + base + 32];
  }
  constexpr int PPT = BN / 64;     // pairs per tile
  if constexpr (EPI == EPI_RESID) {
    a.x[base] += x1;
    a.x[base + 32] += x2;
  } else if constexpr (EPI == EPI_QKV) {
    epi_qkv<BN>(a, row, g / PPT, g % PPT, c, x1, x2);
  } else if constexpr (EPI == EPI_GATE_UP) {
    epi_gate_up<BN>(a, row, g / PPT, g % PPT, c, x1, x2);
  }
}

// Split-K reduction of a residual product fused with the RMSNorm that
// follows it: x += (sum of the splits, in split order), then
// norm_out = bf16(x / sqrt(mean(x^2) + eps) * gain), one 256-thread block per
// row, CPT 4-float chunks of the row per thread (N <= 1024 * CPT).  Bitwise
// the same as splitk_reduce_kernel followed by the stand-alone RMSNorm (same
// summation orders), one pass over the row fewer.  Every chunk's split loads
// are issued together, four splits per round.  EAGER (few rows, so few blocks
// to hide latency with): the residual row is loaded before the splits and
// eight splits go per round, for fewer round trips at the price of registers
// (at 1024 rows the lost occupancy costs more: O 1.78 -> 1.88 ms per step).
template <int CPT, bool EAGER>
__global__ __launch_bounds__(256) void splitk_reduce_norm_kernel(GemmArgs a) {
  __shared__ float red[4];
  const int row = blockIdx.x;
  float* xr = a.x + (size_t)row * a.N;
  const size_t plane = (size_t)a.M * a.N;
  const float* pr = a.partial + (size_t)row * a.N;
  f32x4 v[CPT], t[CPT], x0[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    t[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int c = (threadIdx.x + 256 * k) * 4;
    if (EAGER && c < a.N) x0[k] = *(const f32x4*)(xr + c);   // in flight with the first splits
  }
  int s = 0;
  if constexpr (EAGER && CPT <= 4) {  // eight splits per round while the registers allow
    for (; s + 8 <= a.ksplit; s += 8) {
      f32x4 p[8][CPT];
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int k = 0; k < CPT; ++k) {
          const int c = (threadIdx.x + 256 * k) * 4;
          p[q][k] = c < a.N ? *(const f32x4*)(pr + (s + q) * plane + c) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int k = 0; k < CPT; ++k) t[k] += p[q][k];
    }
  }
  for (; s + 4 <= a.ksplit; s += 4) {
    f32x4 p[4][CPT];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < CPT; ++k) {
        const int c = (threadIdx.x + 256 * k) * 4;
        p[q][k] = c < a.N ? *(const f32x4*)(pr + (s + q) * plane + c) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < CPT; ++k) t[k] += p[q][k];
  }
  for (; s < a.ksplit; ++s)
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = (threadIdx.x + 256 * k) * 4;
      if (c < a.N) t[k] += *(const f32x4*)(pr + s * plane + c);
    }
  float ss = 0.f;
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = (threadIdx.x + 256 * k) * 4;
    if (c < a.N) {
      v[k] = (EAGER ? x0[k] : *(const f32x4*)(xr + c)) + t[k];
      *(f32x4*)(xr + c) = v[k];
      ss += v[k][0] * v[k][0] + v[k][1] * v[k][1] + v[k][2] * v[k][2] + v[k][3] * v[k][3];
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = red[0] + red[1] + red[2] + red[3];
  const float rstd = rsqrtf(tot / (float)a.N + a.norm_eps);
  bf16* orow = a.norm_out + (size_t)row * a.N;
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = (threadIdx.x + 256 * k) * 4;
    if (c < a.N) {
      const bf16x4 g = *(const bf16x4*)(a.norm_gain + c);
      bf16x4 y;
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = (bf16)(v[k][j] * rstd * (float)g[j]);
      *(bf16x4*)(orow + c) = y;
    }
  }
}

// Launch the fused reduction + norm; false when the row is too long for it.
bool launch_reduce_norm(const GemmArgs& a, hipStream_t s) {
  const int cpt = (a.N + 1023) / 1024;
  const bool eager = a.M <= 512;       // at most two blocks per CU
  auto go = [&](auto kern) { kern<<<(unsigned)a.M, 256, 0, s>>>(a); return true; };
  switch (cpt) {
    case 1: return eager ? go(splitk_reduce_norm_kernel<1, true>) : go(splitk_reduce_norm_kernel<1, false>);
    case 2: return eager ? go(splitk_reduce_norm_kernel<2, true>) : go(splitk_reduce_norm_kernel<2, false>);
    case 3:
    case 4: return eager ? go(splitk_reduce_norm_kernel<4, true>) : go(splitk_reduce_norm_kernel<4, false>);
    case 5: case 6: case 7:
    case 8: return eager ? go(splitk_reduce_norm_kernel<8, true>) : go(splitk_reduce_norm_kernel<8, false>);
    default: return false;
  }
}

enum TileShape { TILE_256x256, TILE_256x128, TILE_128x128, TILE_64x256, TILE_32x256 };

struct TilePlan {
  TileShape shape;
  int splits;       // K splits
};

// K splits of the ring kernel's tiles: about one work-group per CU for
// 128 x 128 (its ring holds a CU's LDS) and two for the skinny ones, at least
// 8 K steps per split, the splits dividing the K steps, partials within the
// workspace area.
int ring_splits(int epi, int BM, long tiles, int M, int N, int K) {
  if (epi == EPI_ARGMAX) return 1;
  const long target = BM <= 64 ? 512 : 256;
  int s = (int)std::max<long>(1, std::min<long>(16, target / tiles));
  const int kt = K / 64;
  while (s > 1 && (kt % s != 0 || kt / s < 8 || (size_t)s * M * N * 4 > kPartialCap)) --s;
  return s;
}

// Shape and splits (measured over the verify step's products):
//   * few rows: 32- or 64-row tiles that stream 256 weight rows each;
//   * up to 128 rows, and products too narrow to give 64 256 x 128 tiles over a
//     short K: 128 x 128 tiles with split K;
//   * many rows: 256 x 256 or 256 x 128 tiles, unsplit or with K split, whichever
//     the cost model below puts first.
// 256-wide tiles need every weight segment (q/k/v) to be a multiple of 256 so
// no tile straddles two; 128-wide ones need multiples of 128.
//
// The model, in us: rounds of 256 work-groups, each (K steps x step + fixed),
// plus a reduction that writes and reads the fp32 partials.  The step times are
// those of a full chip (gate/up, 8B shape: 256 x 256 at 1024 rows 213 us over
// 2 x 64 steps, 256 x 128 at 4096 rows 824 us over 14 x 64).  Measured us
// against the form that is not taken, 8B shape, reduction included:
//   1024 rows: down 256x256 split 4 118, 256x128 split 2 125; O 256x128 split 2
//   50, 256x256 split 4 53; q/k/v 256x128 64, 256x256 split 2 76;
//   512 rows: gate/up 256x256 106, 256x128 121; down 256x128 split 4 70,
//   256x256 split 4 88; O 256x128 split 4 32, split 2 39;
//   200 rows: gate/up 256x128 65, 256x256 80.
TilePlan pick_tile(int epi, int M, int N, int K, int n0, int n1, bool may_split) {
  const bool w256 = N % 256 == 0 && n0 % 256 == 0 && n1 % 256 == 0;
  auto ring = [&](TileShape t, int BM, int BN) {
    const long tiles = (long)((M + BM - 1) / BM) * (N / BN);
    return TilePlan{t, may_split ? ring_splits(epi, BM, tiles, M, N, K) : 1};
  };
  if (w256 && M <= 32) return ring(TILE_32x256, 32, 256);
  if (w256 && M <= 64) return ring(TILE_64x256, 64, 256);
  const long mt = (M + 255) / 256;
  if (M <= 128 || (mt * (N / 128) < 64 && K <= 4096)) return ring(TILE_128x128, 128, 128);
  const int kt = K / 64;
  TilePlan best{TILE_256x128, 1};
  double best_us = 1e30;
  for (const TileShape t : {TILE_256x256, TILE_256x128}) {
    if (t == TILE_256x256 && !w256) continue;
    const long tiles = mt * (N / (t == TILE_256x256 ? 256 : 128));
    const double step = t == TILE_256x256 ? 1.55 : 0.95;
    for (int s = 1; s <= (may_split && epi != EPI_ARGMAX ? 16 : 1); ++s) {
      if (s > 1 && (kt % s != 0 || kt / s < 8 || (size_t)s * M * N * 4 > kPartialCap)) continue;
      if (t == TILE_256x256 && (kt / s) % 2 != 0) continue;     // its steps go in pairs
      const double rounds = (double)((tiles * s + 255) / 256);
      double us = rounds * (kt / s * step + 5.0);
      if (s > 1) us += 4.0 + 8.0 * s * M * N / 4.5e6;
      if (us < best_us) {
        best_us = us;
        best = TilePlan{t, s};
      }
    }
  }
  return best;
}

// Sum the splits and apply the epilogue of a product on BN-wide tiles.
template <int EPI, int BN>
hipError_t launch_reduce(const GemmArgs& a, hipStream_t s) {
  if (EPI == EPI_RESID && a.norm_out != nullptr && a.N % 4 == 0 && launch_reduce_norm(a, s)) {
    if (a.norm_done) *a.norm_done = true;
  } else {
    const size_t threads = (size_t)a.M * (a.N / 2);
    splitk_reduce_kernel<EPI, BN><<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(a);
  }
  return hipGetLastError();
}

template <int EPI, int BM, int BN, int THREADS, int SMEM, class Kernel>
hipError_t launch_tiles(Kernel kernel, const GemmArgs& a, hipStream_t s) {
  static bool configured = false;
  if (!configured) {
    const hipError_t e =
        hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const long tiles = (long)((a.M + BM - 1) / BM) * (a.N / BN);
  kernel<<<(unsigned)(tiles * a.ksplit), THREADS, SMEM, s>>>(a);
  return a.ksplit > 1 ? launch_reduce<EPI, BN>(a, s) : hipGetLastError();
}

template <int EPI, int BM, int BN, int WM, int NS>
hipError_t launch_ring(const GemmArgs& a, hipStream_t s) {
  return launch_tiles<EPI, BM, BN, 256, NS * (BM + BN) * 128>(gemm_ring_kernel<EPI, BM, BN, WM, NS>, a, s);
}

template <int EPI>
hipError_t launch_epi(GemmArgs a, hipStream_t s) {
  // Few rows: every supported shape has K a multiple of 128 and head_dim 64
  // or 128, which the weight-row units assume.
  if constexpr (EPI != EPI_ARGMAX)
    if (a.M <= skinny_max_rows<EPI>() && a.K % 128 == 0) return launch_skinny<EPI>(a, s);
  const TilePlan p = pick_tile(EPI, a.M, a.N, a.K, a.n0, a.n1, a.partial != nullptr);
  a.ksplit = p.splits;
  switch (p.shape) {
    case TILE_256x256:
      return launch_tiles<EPI, 256, 256, 512, 2 * 512 * 128>(gemm_256x256_kernel<EPI>, a, s);
    case TILE_256x128:
      return launch_tiles<EPI, 256, 128, 512, 3 * 384 * 128>(gemm_256x128_kernel<EPI>, a, s);
    case TILE_32x256: return launch_ring<EPI, 32, 256, 1, 3>(a, s);
    case TILE_64x256: return launch_ring<EPI, 64, 256, 2, 3>(a, s);
    default: return launch_ring<EPI, 128, 128, 2, 4>(a, s);
  }
}

}  // namespace

int gemm_parts(int N, int M, int K) {
  switch (pick_tile(EPI_ARGMAX, M, N, K, N, 0, false).shape) {
    case TILE_64x256: return N / 128;
    default: return N / 64;       // all others: wave slabs of 64 columns
  }
}

size_t gemm_partial_bytes() { return kPartialCap; }

hipError_t launch_gemm(int epi, const GemmArgs& a, hipStream_t s) {
  switch (epi) {
    case EPI_QKV: return launch_epi<EPI_QKV>(a, s);
    case EPI_RESID: return launch_epi<EPI_RESID>(a, s);
    case EPI_GATE_UP: return launch_epi<EPI_GATE_UP>(a, s);
    case EPI_ARGMAX: return launch_epi<EPI_ARGMAX>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace spec
