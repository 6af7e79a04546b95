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
// The kernels (plan_gemm() chooses; each has its own comment):
//   * gemm_256x256_kernel, gemm_256x128_kernel: many rows, two wave groups in
//     opposite phases;
//   * gemm_ring_kernel: 64 x 64, 64 x 128 and 128 x 128 tiles, for products
//     whose weights are streamed;
//   * few_rows_gemm_kernel: gate/up and q/k/v of up to 4 rows.
// The tile kernels share their operand path: tiles move HBM/L2 -> LDS with
// global_load_lds_dwordx4 (no register staging) into stages of 64 K columns,
// later stages in flight while one is multiplied (vmcnt counts them out, so a
// barrier never waits for the whole ring).  Each wave-load writes 1 KB = 8
// tile rows of 128 bytes; the 16-byte chunk index of row r is XOR-ed with
// (r >> 1) & 7, which makes the MFMA operand reads (16 consecutive rows, one
// chunk) hit all 64 LDS banks once.
//
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

typedef __attribute__((address_space(3))) char lds_char;

// Direct global -> LDS load of 16 bytes per lane from base + voff to the
// wave-uniform LDS address `lds` + 16 * lane.  In assembly, so that the
// compiler does not wait for it at the next LDS read; the kernels' own vmcnt
// waits and barriers order it.  The s_nop is the wait state that the load needs
// after a write of M0.
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
               : "memory", "m0");
}

// Barrier that no memory access and no instruction is moved across.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// 16-byte chunk swizzle of tile row `row` (rows of 128 bytes): 16 consecutive
// rows reading one logical chunk hit 16 distinct 16-byte bank groups.
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// Wait until at most N vector-memory operations of this wave are in flight.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Virtual columns: every group of 64 is one pair of 32-column blocks, the
// members of pair `v / 64`: rotary partners (dims j, j + d/2) of one head, or
// (gate, up) of one feature.  A segment (q, k, v) is a whole number of groups.
struct QkvColumn {
  int seg;        // 0 q, 1 k, 2 v
  int head;       // head of the segment
  int freq0;      // first rotary frequency (first member's dim) of the group
};
__device__ __forceinline__ QkvColumn qkv_group(const GemmArgs& a, int v) {
  QkvColumn q;
  q.seg = v < a.n0 ? 0 : (v < a.n0 + a.n1 ? 1 : 2);
  const int local = (v - (q.seg == 0 ? 0 : (q.seg == 1 ? a.n0 : a.n0 + a.n1))) >> 6, qpd = a.head_dim / 64;
  q.head = local / qpd;
  q.freq0 = (local % qpd) * 32;
  return q;
}

// Weight row of virtual column v.
template <int EPI>
__device__ __forceinline__ const bf16* weight_row(const GemmArgs& a, int v) {
  const int blk = (v >> 5) & 1, c = v & 31;
  if constexpr (EPI == EPI_QKV) {
    const QkvColumn q = qkv_group(a, v);
    const bf16* base = q.seg == 0 ? a.B0 : (q.seg == 1 ? a.B1 : a.B2);
    return base + (size_t)(q.head * a.head_dim + q.freq0 + blk * (a.head_dim / 2) + c) * a.K;
  } else if constexpr (EPI == EPI_GATE_UP) {
    return (blk ? a.B1 : a.B0) + (size_t)((v >> 6) * 32 + c) * a.K;
  } else {
    return a.B0 + (size_t)v * a.K;
  }
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }

// Pair epilogues of the split-K reduction: (x1, x2) are the two members of the
// pair of 64-column group g, lane column c, output row `row`.
__device__ __forceinline__ void epi_qkv(const GemmArgs& a, int row, int g, int c, float x1, float x2) {
  const QkvColumn q = qkv_group(a, g * 64);
  const int hd = a.head_dim, half = hd / 2, fi = q.freq0 + c;
  if (q.seg < 2) {
    const float2 cs = a.rope_cs[(size_t)row * half + fi];
    const float y1 = x1 * cs.x - x2 * cs.y;
    const float y2 = x2 * cs.x + x1 * cs.y;
    x1 = y1;
    x2 = y2;
  }
  if (q.seg == 0) {
    bf16* pq = a.q_out + (size_t)row * a.n0 + q.head * hd + fi;
    pq[0] = (bf16)x1;
    pq[half] = (bf16)x2;
  } else {
    const TokInfo t = a.toks[row];
    const SampleInfo s = a.samples[t.sample];
    const int slot = s.seq_len + t.node;
    bf16* pk = a.kv_pool + s.kv_base +
               ((((size_t)a.layer * 2 + (q.seg - 1)) * a.n_kv_heads + q.head) * s.cap + slot) * hd + fi;
    pk[0] = (bf16)x1;
    pk[half] = (bf16)x2;
  }
}

__device__ __forceinline__ void epi_gate_up(const GemmArgs& a, int row, int g, int c, float gate, float up) {
  a.act_out[(size_t)row * (a.N / 2) + g * 32 + c] = (bf16)(silu(gate) * up);
}

// Work-group b runs on XCD b % 8, which receives q + 1 work-groups (x < r)
// or q (x >= r) for a grid of 8q + r.  Give each XCD a contiguous range of
// logical ids, so that the M tiles sharing a weight tile (adjacent ids)
// meet in one XCD's L2.
__device__ __forceinline__ int xcd_contiguous(int b, int total) {
  const int q = total >> 3, r = total & 7, x = b & 7, j = b >> 3;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
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

// The epilogues.  The products are taken as D = W . A^T, so a lane's four
// accumulators of a 16 x 16 block are four consecutive output columns of one
// row: acc[i][j][e] = row 16 i + lane % 16, column 16 j + 4 (lane / 16) + e of
// the wave's tile, and every output goes out as 8 or 16 bytes per lane.  The
// wave's tile starts at row row0 and column col0 (a
// multiple of 64) of tile (tm, tn); blocks j and j + 2 (j = 0, 1) hold the pairs of weight_row().
template <int EPI, int BM, int BN, int MB, int NB>
__device__ __forceinline__ void epilogue_rows(const GemmArgs& a, f32x4 (&acc)[MB][NB], int tm, int tn,
                                              int row0, int col0, int split, int lane) {
  const int m = tm * BM + row0 + (lane & 15), c4 = 4 * (lane >> 4);
  if (a.plan.splits > 1) {      // raw fp32 tile of this split, virtual column order
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
    constexpr int RP = MB < 2 ? 1 : 2;       // rows whose residuals are in flight together
#pragma unroll
    for (int i0 = 0; i0 < MB; i0 += RP) {
      f32x4 xv[RP][NB];
#pragma unroll
      for (int i = 0; i < RP; ++i) {
        const int row = m + 16 * (i0 + i);
        if (row < a.M)
#pragma unroll
          for (int j = 0; j < NB; ++j) xv[i][j] = *(const f32x4*)(x + (size_t)row * a.N + 16 * j);
      }
#pragma unroll
      for (int i = 0; i < RP; ++i) {
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
    const QkvColumn q = qkv_group(a, tn * BN + col0);
    const int seg = q.seg, head = q.head, hd = a.head_dim, half = hd / 2, fi = q.freq0 + c4;
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

// ---- many rows: 256-row tiles, two wave groups in opposite phases ---------
//
// Both kernels below run 8 waves, two per SIMD, as two groups of four (group g
// = wave / 4; waves w and w + 4 share a SIMD).  A K step is cut into phases,
// each a memory part (fragment reads from LDS, direct loads of a later K step)
// and an MFMA part, separated by work-group barriers; group 1 runs one barrier
// behind group 0, so on every SIMD one wave's MFMAs always meet the other
// wave's memory part and the matrix core does not wait for LDS.  (In a plain ring
// all waves read, then all multiply.)  Measured on the gate/up
// product of the 8B shape (28672 x 4096, weights from HBM), us at 512 / 1024 /
// 4096 rows: plain ring 150 / 253 / 878, these phases with the same 32x32x16
// instructions 124 / 232 / 768.  The clock then falls with the load (counters
// over the whole kernel at 4096 rows: 1.8 of 2.4 GHz, the matrix cores busy in
// 83 % of its cycles; presumably the card's power limit), so energy per product
// counts: 16x16x32 instructions, whose accumulator traffic per flop is half,
// sustain 2.06 against 1.83 PFLOP/s in a loop of MFMAs alone, and take the same
// product to 106 / 213 / 699 us (1.38 PFLOP/s at 4096 rows; 634 to 699 from one
// card to another).

// 256 x 256 tiles, 64-wide K steps in two stages of 64 KB.  Group g holds rows
// 128 g .., wave q = wave % 4 of it columns 64 q ..: 128 x 64 per wave.  Every
// step is four phases of 16 MFMAs, one quadrant (64 rows x 32 columns, K = 64)
// each: (A0, B0), (A0, B1), (A1, B1), (A1, B0), A0 / A1 the halves of the
// wave's rows and B0 / B1 of its columns.  A half is read into registers once,
// B0 of the next step in the last phase, so the LDS rows of a half are free one
// phase after their read and take the step after next: phases 0 .. 3 load A1
// (next step), B0, A0, B1 (step after next), two wave-loads per wave each, and
// every load has five phases (of 512 MFMA cycles, both groups') to arrive.  Group 1's
// reads of phase p are complete at the barrier that ends its phase, and group 0
// is then still in phase p + 1; B0 of step 0, read in front of phase 0 and
// refilled in phase 1, is waited for where it is read.
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
  const int KT = a.K / 64 / a.plan.splits;            // K steps of this split (even)
  const size_t k_off = (size_t)split * KT * 64;

  // Wave-load j of half hh: 8 tile rows of 128 bytes; lane l lands at row l / 8,
  // chunk l % 8, so it fetches logical chunk (l % 8) ^ swz(row).
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t va[2][2], vb[2][2], la[2][2], lb[2][2];
  const int mlast = a.M - 1 - tm * BM;           // rows past M repeat the last row; never stored
  const bf16* abase = a.A + (size_t)tm * BM * a.K + k_off;
  const bf16* bbase[2] = {weight_row<EPI>(a, tn * BN) + k_off, weight_row<EPI>(a, tn * BN + 32) + k_off};
#pragma unroll
  for (int hh = 0; hh < 2; ++hh)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int c = wave * 2 + j;
      const int ra = (c >> 3) * 128 + hh * 64 + (c & 7) * 8, rb = (c >> 2) * 64 + hh * 32 + (c & 3) * 8;
      va[hh][j] = (uint32_t)min(ra + lr, mlast) * a.K * 2 + ((lc ^ swz(ra + lr)) << 4);
      vb[hh][j] = (uint32_t)((const char*)(weight_row<EPI>(a, tn * BN + rb + lr) + k_off) - (const char*)bbase[hh]) +
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
  wait_lds();                                    // step 0 refills these rows one phase early
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
  const int KT = a.K / 64 / a.plan.splits;            // at least 2
  const size_t k_off = (size_t)split * KT * 64;

  // Wave-loads as above: wave w loads A rows 32 w .. and weight rows 16 w ..
  // (which lie in one 32-row block, of one weight matrix).
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t va[4], vb[2];
  const int mlast = a.M - 1 - tm * BM;
  const bf16* abase = a.A + (size_t)tm * BM * a.K + k_off;
  const bf16* bbase = weight_row<EPI>(a, tn * BN + (wave >> 1) * 32) + k_off;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ra = (wave * 4 + j) * 8 + lr;
    va[j] = (uint32_t)min(ra, mlast) * a.K * 2 + ((lc ^ swz(ra)) << 4);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int rb = (wave * 2 + j) * 8 + lr;
    vb[j] = (uint32_t)((const char*)(weight_row<EPI>(a, tn * BN + rb) + k_off) - (const char*)bbase) +
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
  // The reads are complete before the barrier: the other group may refill the
  // stage right after it.
  auto multiply = [&]() {
    wait_lds();
    phase_barrier();
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

// ---- the ring kernel: products whose weights are streamed -------------------
//
// BM x BN tiles on 4 waves, each BM / WM x 64 in a WM x BN/64 grid, NS stages.
// Up to some 256 rows a product is bound by the bytes its CUs can take in: the
// weights from HBM (about 6 TB/s) and, as often as there are weight tiles, the
// rows from L2 (about 13 TB/s over the chip), so the tile is chosen for the
// fewest of both with every CU loading: 64 x 64 for narrow products (8B O and
// down, all of 1B's, up to 64 rows; its 64 KB leave two work-groups on a CU, each
// covering the other's waits), 64 x 128 (72 KB, also two) for wide ones (8B q/k/v
// and gate/up from 5 rows) and 128 x 128 (128 KB, one) beyond 64 rows.  Deeper rings, and rings in
// which some waves load only rows and the others only weights, were no faster.
// An unsplit product starts its K loop at a step that depends on the weight
// tile (and wraps around): with all CUs at the same K of rows 2^n bytes apart
// the loads meet in a few HBM channels (8B gate/up at 64 rows 49.3 -> 43.7 us =
// 5.4 TB/s of weights, 1B gate/up 17.8 -> 14.8); K splits are spread already.
// Measured against 32 x 256 and 64 x 256 tiles with 32x32x16 instructions, us
// with the split-K reduction, 8B shape at 16 / 64 rows: gate/up 47.3 -> 42.7 /
// 57.4 -> 43.8; down with its norm 30.5 -> 27.4 / 33.3 -> 30.0; O with its norm
// 15.9 -> 13.3 / 18.6 -> 14.4; q/k/v 16.1 -> 14.1 / 19.3 -> 16.5.
template <int EPI, int BM, int BN, int NS>
__global__ __launch_bounds__(256) void gemm_ring_kernel(GemmArgs a) {
  constexpr int WN = BN / 64, WM = 4 / WN, MB = BM / WM / 16;
  constexpr int ROWB = 128, STAGE = (BM + BN) * ROWB, BOFF = BM * ROWB;
  constexpr int AL = BM / 32, BL = BN / 32;      // wave-loads per wave and stage
  static_assert(MB >= 1 && (NS - 2) * (AL + BL) <= 63, "tile shape");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int ntm = (a.M + BM - 1) / BM, ntn = a.N / BN, tiles = ntm * ntn;
  const int bid = xcd_contiguous(blockIdx.x, gridDim.x);
  const int split = bid / tiles;
  int tm, tn;
  tile_at(bid % tiles, ntm, ntn, &tm, &tn);
  const int KT = a.K / 64 / a.plan.splits;            // K steps of this split
  const size_t k_off = (size_t)split * KT * 64;

  // Wave w loads A rows 8 AL w .. and weight rows 8 BL w .. (at most 32, which
  // lie in one 32-column block, of one weight matrix).
  const int lr = lane >> 3, lc = lane & 7;
  uint32_t va[AL], vb[BL];
  const int mlast = a.M - 1 - tm * BM;           // rows past M repeat the last row; never stored
  const bf16* abase = a.A + (size_t)tm * BM * a.K + k_off;
  const bf16* bbase = weight_row<EPI>(a, tn * BN + wave * BL * 8) + k_off;
#pragma unroll
  for (int j = 0; j < AL; ++j) {
    const int ra = (wave * AL + j) * 8 + lr;
    va[j] = (uint32_t)min(ra, mlast) * a.K * 2 + ((lc ^ swz(ra)) << 4);
  }
#pragma unroll
  for (int j = 0; j < BL; ++j) {
    const int rb = (wave * BL + j) * 8 + lr;
    vb[j] = (uint32_t)((const char*)(weight_row<EPI>(a, tn * BN + rb) + k_off) - (const char*)bbase) +
            ((lc ^ swz(rb)) << 4);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
  const uint32_t lds_a = lds0 + wave * AL * 1024, lds_b = lds0 + BOFF + wave * BL * 1024;
  const int rot = a.plan.splits == 1 ? tn * 5 % KT : 0;
  auto load = [&](int kt, uint32_t st) {
    const int k = kt + rot < KT ? kt + rot : kt + rot - KT;
    const char* bs = (const char*)bbase + (size_t)k * ROWB;
    const char* as = (const char*)abase + (size_t)k * ROWB;
#pragma unroll
    for (int j = 0; j < BL; ++j) dma16(bs, vb[j], lds_b + st + j * 1024);
#pragma unroll
    for (int j = 0; j < AL; ++j) dma16(as, va[j], lds_a + st + j * 1024);
  };

  f32x4 acc[MB][4];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};
  const int r = lane & 15;
  uint32_t ro[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) ro[ks] = r * ROWB + (((4 * ks + (lane >> 4)) ^ swz(r)) << 4);
  const char* arows = smem + wm * (BM / WM) * ROWB;
  const char* brows = smem + BOFF + wn * 64 * ROWB;

#pragma unroll
  for (int k = 0; k < NS - 1; ++k)
    if (k < KT) load(k, k * STAGE);
  uint32_t st = 0, fill = (NS - 1) * STAGE;      // stage being read, stage being filled
  for (int kt = 0; kt < KT; ++kt) {
    // Stage kt has landed for every wave after the barrier (later stages may be
    // in flight), and every wave's reads of stage kt - 1 are complete (its MFMAs
    // are issued): that stage is refilled.
    if (kt + NS - 2 < KT) wait_vm<(NS - 2) * (AL + BL)>();
    else wait_vm<0>();
    phase_barrier();
    if (kt + NS - 1 < KT) load(kt + NS - 1, fill);
    bf16x8 fa[2][MB], fb[2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[ks][i] = *(const bf16x8*)(arows + st + i * 16 * ROWB + ro[ks]);
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[ks][j] = *(const bf16x8*)(brows + st + j * 16 * ROWB + ro[ks]);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    st = st == (NS - 1) * STAGE ? 0 : st + STAGE;
    fill = fill == (NS - 1) * STAGE ? 0 : fill + STAGE;
  }
  epilogue_rows<EPI, BM, BN, MB, 4>(a, acc, tm, tn, wm * (BM / WM), wn * 64, split, lane);
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
// epilogue; no K split leaves the work-group, so no reduction kernel follows.
// Units: QKV = 8 rotary pairs (dims j, j + d/2) of one head, GATE_UP = 8
// (gate, up) features.  Every unit reads all M activation rows, so the
// activation bytes grow with M against a fixed weight stream.  Whole steps of 8
// layers, with these two products here or on tiles: 8B at 4 rows 1105 or 1108
// us, at 8 rows 1189 or 1117.  The residual products do not come here, as a K
// split's reduction takes their RMSNorm with it (one row, with the norm: down
// 28.7 on tiles, 30.8 here, O 13.4 and 14.7; the 1B step of 8 layers 520 and 550).  Accumulator layout of the 16 x 16
// block: lane l, element i holds activation row 4 (l / 16) + i and unit row
// l % 16.
constexpr int kUnitRows = 16;
constexpr int kFewRows = 4;          // activation rows up to which a product comes here

template <int EPI>
__device__ __forceinline__ const bf16* unit_row(const GemmArgs& a, int unit, int c) {
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
  } else {
    const int f = unit * 8 + (c & 7);
    return (c < 8 ? a.B0 : a.B1) + (size_t)f * a.K;
  }
}

template <int EPI>
__global__ __launch_bounds__(256) void few_rows_gemm_kernel(GemmArgs a) {
  static_assert(EPI == EPI_QKV || EPI == EPI_GATE_UP, "a product of pairs");
  __shared__ f32x4 red[4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, kq = lane >> 4;
  const int unit = blockIdx.x;
  const int kw = a.K / 4;                            // K of this wave (a multiple of 32)
  const int k0 = wave * kw, k1 = k0 + kw;
  const bf16* wrow = unit_row<EPI>(a, unit, c) + kq * 8;
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
    if constexpr (EPI == EPI_GATE_UP) {
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
hipError_t launch_few_rows(const GemmArgs& a, hipStream_t s) {
  const long grid = (long)a.N / kUnitRows;
  few_rows_gemm_kernel<EPI><<<(unsigned)grid, 256, 0, s>>>(a);
  return hipGetLastError();
}

// Sum the K splits in split order and apply the epilogue.  Thread (row,
// group g of 64 virtual columns, lane column c) owns virtual columns g*64 + c
// and g*64 + 32 + c: a pair, or two residual columns.
template <int EPI>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int half_n = a.N / 2;
  if (idx >= (size_t)a.M * half_n) return;
  const int row = (int)(idx / half_n), rem = (int)(idx % half_n);
  const int g = rem >> 5, c = rem & 31;
  const size_t base = (size_t)row * a.N + g * 64 + c;
  float x1 = 0.f, x2 = 0.f;
  for (int s = 0; s < a.plan.splits; ++s) {
    x1 += a.partial[(size_t)s * a.M * a.N + base];
    x2 += a.partial[(size_t)s * a.M * a.N + base + 32];
  }
  if constexpr (EPI == EPI_RESID) {
    a.x[base] += x1;
    a.x[base + 32] += x2;
  } else if constexpr (EPI == EPI_QKV) {
    epi_qkv(a, row, g, c, x1, x2);
  } else if constexpr (EPI == EPI_GATE_UP) {
    epi_gate_up(a, row, g, c, x1, x2);
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
    for (; s + 8 <= a.plan.splits; s += 8) {
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
  for (; s + 4 <= a.plan.splits; s += 4) {
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
  for (; s < a.plan.splits; ++s)
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

// Sum the splits and apply the epilogue.
template <int EPI>
hipError_t launch_reduce(const GemmArgs& a, hipStream_t s) {
  if (EPI == EPI_RESID && a.norm_out != nullptr && a.N % 4 == 0 && launch_reduce_norm(a, s)) {
    if (a.norm_done) *a.norm_done = true;
  } else {
    const size_t threads = (size_t)a.M * (a.N / 2);
    splitk_reduce_kernel<EPI><<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(a);
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
  kernel<<<(unsigned)(tiles * a.plan.splits), THREADS, SMEM, s>>>(a);
  return a.plan.splits > 1 ? launch_reduce<EPI>(a, s) : hipGetLastError();
}

template <int EPI, int BM, int BN, int NS>
hipError_t launch_ring(const GemmArgs& a, hipStream_t s) {
  return launch_tiles<EPI, BM, BN, 256, NS * (BM + BN) * 128>(gemm_ring_kernel<EPI, BM, BN, NS>, a, s);
}

template <int EPI>
hipError_t launch_epi(const GemmArgs& a, hipStream_t s) {
  if constexpr (EPI == EPI_QKV || EPI == EPI_GATE_UP)
    if (a.plan.shape == GEMM_FEW_ROWS) return launch_few_rows<EPI>(a, s);
  switch (a.plan.shape) {
    case GEMM_256x256:
      return launch_tiles<EPI, 256, 256, 512, 2 * 512 * 128>(gemm_256x256_kernel<EPI>, a, s);
    case GEMM_256x128:
      return launch_tiles<EPI, 256, 128, 512, 3 * 384 * 128>(gemm_256x128_kernel<EPI>, a, s);
    case GEMM_128x128: return launch_ring<EPI, 128, 128, 4>(a, s);
    case GEMM_64x128: return launch_ring<EPI, 64, 128, 3>(a, s);
    case GEMM_64x64: return launch_ring<EPI, 64, 64, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// The cost model, in us: the larger of the weight stream (6.1 TB/s) and of the
// work-groups' own time, an eighth of the smaller, which overlaps imperfectly,
// and for a split the reduction (3.3 + 0.1 per split + its fp32 partials, written
// and read, at 6 TB/s).  A work-group's K step of 64 takes `step` with the chip
// full; the 64-row tiles run two to a CU, whose pair takes `pair` steps, and the
// others' step shrinks to `alone` of it when few CUs work (less L2 traffic, and a
// higher clock).  `fixed` is each round's prologue and epilogue.  An unsplit
// residual product leaves its RMSNorm to a launch of its own (5 us); a reduction
// takes it along.  Launched back to back on the 8B and 1B shapes' products, 1 to
// 4096 rows, weights from HBM, the five tiles and their splits (3285 times taken)
// need about 3 us a launch more than the model says (17 % rms; 9 % with the 3 us
// added), and the one chosen is on average 1.0 % slower than the best of them, at
// worst 18 % (1B O at 640 rows, 22.1 against 18.7 us).  Storing the logits has no
// term (8B head at 1024 rows 751 -> 841 us): with it the choice is 0.3 % off.
GemmPlan plan_gemm(int epi, int M, int N, int K, int n0, int n1, bool norm) {
  if ((epi == EPI_QKV || epi == EPI_GATE_UP) && M <= kFewRows) return GemmPlan{GEMM_FEW_ROWS, 1};
  // LM head of few rows: the model puts 64 x 64 and 64 x 128 tiles level.  Whole
  // steps with either, us: 8B, 4 layers, 641 or 649 at 4 rows, 661 or 671 at 16,
  // 674 or 683 at 32, 702 or 709 at 48, 738 or 736 at 64, 915 or 888 at 96; 1B, 8
  // layers, level to 48 rows (595 or 594 at 32), 661 or 654 at 64, 801 or 786 at 96.
  if (epi == EPI_ARGMAX && M <= 32) return GemmPlan{GEMM_64x64, 1};
  struct Tile {
    GemmShape shape;
    int bm, bn;
    double step, pair, alone, fixed;
  };
  static constexpr Tile tiles[] = {{GEMM_256x256, 256, 256, 1.319, 0, 0.705, 3.17},
                                   {GEMM_256x128, 256, 128, 0.822, 0, 0.769, 2.06},
                                   {GEMM_128x128, 128, 128, 0.626, 0, 0.854, 1.45},
                                   {GEMM_64x128, 64, 128, 0.449, 1.607, 1, 0.39},
                                   {GEMM_64x64, 64, 64, 0.281, 1.776, 1, 0.25}};
  const int kt = K / 64;
  const double stream = 2e-6 * N * K / 6.1;
  GemmPlan best{GEMM_128x128, 1};
  double best_us = 1e30;
  for (const Tile& t : tiles) {
    // A 256-wide tile addresses its weight rows from one base per block parity,
    // so it needs segments (q/k/v) that are multiples of 256; its K steps go in
    // pairs.  Every supported width is a multiple of 128.
    if (t.bn == 256 && (N % 256 || n0 % 256 || n1 % 256)) continue;
    const long count = (long)((M + t.bm - 1) / t.bm) * (N / t.bn);
    for (int s = 1; s <= (epi == EPI_ARGMAX ? 1 : 16); ++s) {
      if (s > 1 && (kt % s != 0 || kt / s < 4 || (size_t)s * M * N * 4 > kPartialCap)) continue;
      if (t.bn == 256 && (kt / s) % 2 != 0) continue;
      const long wgs = count * s;
      const int per = t.pair > 0 ? 512 : 256;            // work-groups of a round
      const double full = t.pair > 0 ? t.pair : 1;       // steps a full round takes
      double rounds, steps;
      if (wgs > 1536) {
        rounds = (double)wgs / per;
        steps = rounds * full;
      } else {
        const long rest = wgs % per;
        rounds = (double)((wgs + per - 1) / per);
        steps = wgs / per * full + (rest > 256 ? full : rest > 0 ? 1 : 0);
      }
      const double step = t.step * (t.alone + (1 - t.alone) * std::min(1.0, wgs / 256.0));
      const double work = kt / s * step * steps + rounds * t.fixed;
      double us = std::max(stream, work) + 0.13 * std::min(stream, work);
      if (s > 1) us += 3.3 + 0.1 * s + 8e-6 * s * M * N / 6;
      else if (norm) us += 5.0;
      if (us < best_us) {
        best_us = us;
        best = GemmPlan{t.shape, s};
      }
    }
  }
  return best;
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
