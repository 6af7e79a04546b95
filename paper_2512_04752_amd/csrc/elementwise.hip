// The small kernels of the verify step: tree metadata, what a row needs before
// the first layer (rotary angles, embedding, first RMSNorm), RMSNorm, the final
// argmax reduction, greedy tree acceptance and KV compaction.
#include <math.h>

#include <type_traits>

#include "common.h"

namespace spec {

namespace {

// Depth, position and ancestor set of every node: one work-group per sample,
// thread i = node i (a tree has at most kMaxTree nodes).  The set is
// kAncWords 64-bit words, bit t % 64 of word t / 64 standing for node t.
// Pointer jumping: node i holds the set of its ancestors at distance < 2^r
// and its ancestor at distance 2^r (the root points at itself); each round
// publishes both in LDS and takes "set |= set of that ancestor, jump to its
// jump", so ceil(log2 T) rounds cover every depth below T.  Depth is the
// set's size minus one.
__global__ __launch_bounds__(kMaxTree) void tree_meta_kernel(const SampleInfo* samples,
                                                             const int32_t* parents, TokInfo* toks,
                                                             uint64_t* anc, int32_t* dbg_depth,
                                                             int32_t* dbg_pos, uint64_t* dbg_anc) {
  __shared__ uint64_t sset[kMaxTree][kAncWords];
  __shared__ int sjump[kMaxTree];
  const int b = blockIdx.x, i = threadIdx.x;
  const SampleInfo s = samples[b];
  const bool live = i < s.ntok;
  int jump = (live && i > 0) ? parents[s.tok0 + i] : i;
  uint64_t set[kAncWords];
#pragma unroll
  for (int w = 0; w < kAncWords; ++w) set[w] = w == (i >> 6) ? 1ull << (i & 63) : 0ull;
  for (int r = 0; (1 << r) < s.ntok; ++r) {     // same bound in every thread of the sample
#pragma unroll
    for (int w = 0; w < kAncWords; ++w) sset[i][w] = set[w];
    sjump[i] = jump;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kAncWords; ++w) set[w] |= sset[jump][w];
    jump = sjump[jump];
    __syncthreads();
  }
  if (!live) return;
  int size = 0;
#pragma unroll
  for (int w = 0; w < kAncWords; ++w) size += __popcll(set[w]);
  const int row = s.tok0 + i, depth = size - 1;
  toks[row] = TokInfo{b, i, s.seq_len + depth, depth};
#pragma unroll
  for (int w = 0; w < kAncWords; ++w) {
    anc[(size_t)row * kAncWords + w] = set[w];
    if (dbg_anc) dbg_anc[(size_t)row * kAncWords + w] = set[w];
  }
  if (dbg_depth) dbg_depth[row] = depth;
  if (dbg_pos) dbg_pos[row] = s.seq_len + depth;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// Sum of `ss` over a 256-thread block: the lanes, then the four waves in order.
__device__ __forceinline__ float block_sum(float ss, float* red) {
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// Where a row to be normalised comes from: the residual stream, or the
// embedding table, whose row is then also written to the residual stream.
struct ResidualRow {
  const float* x;
  __device__ __forceinline__ f32x4 load(int c) const { return *(const f32x4*)(x + c); }
};
struct EmbeddedRow {
  const bf16* table;
  float* x;
  __device__ __forceinline__ f32x4 load(int c) const {
    const bf16x4 e = *(const bf16x4*)(table + c);
    const f32x4 v = {(float)e[0], (float)e[1], (float)e[2], (float)e[3]};
    *(f32x4*)(x + c) = v;
    return v;
  }
};

// out = bf16(x / sqrt(mean(x^2) + eps) * gain), one 256-thread block per row.
// CPT > 0: the row is CPT 4-element chunks per thread (hidden <= 1024 * CPT),
// all loaded (with their gains) before any is used, so a short row costs one
// memory round trip (with few rows there are few blocks to hide latency);
// CPT = 0: any length, a strided loop.  Both sum each thread's chunks in
// column order, then the lanes, then the four waves: the same result.
template <int CPT, class Row>
__device__ __forceinline__ void normalise_row(const Row& row, const bf16* gain, bf16* orow, int hidden,
                                              float eps, float* red) {
  float ss = 0.f;
  if constexpr (CPT > 0) {
    f32x4 v[CPT];
    bf16x4 g[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = (threadIdx.x + 256 * k) * 4;
      if (c < hidden) {
        v[k] = row.load(c);
        g[k] = *(const bf16x4*)(gain + c);
      }
    }
#pragma unroll
    for (int k = 0; k < CPT; ++k)
      if ((threadIdx.x + 256 * k) * 4 < hidden)
        ss += v[k][0] * v[k][0] + v[k][1] * v[k][1] + v[k][2] * v[k][2] + v[k][3] * v[k][3];
    const float rstd = rsqrtf(block_sum(ss, red) / (float)hidden + eps);
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      const int c = (threadIdx.x + 256 * k) * 4;
      if (c < hidden) {
        bf16x4 y;
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = (bf16)(v[k][j] * rstd * (float)g[k][j]);
        *(bf16x4*)(orow + c) = y;
      }
    }
  } else {
    for (int c = threadIdx.x * 4; c < hidden; c += 256 * 4) {
      const f32x4 v = row.load(c);
      ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
    const float rstd = rsqrtf(block_sum(ss, red) / (float)hidden + eps);
    for (int c = threadIdx.x * 4; c < hidden; c += 256 * 4) {
      const f32x4 v = row.load(c);
      const bf16x4 g = *(const bf16x4*)(gain + c);
      bf16x4 y;
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = (bf16)(v[k] * rstd * (float)g[k]);
      *(bf16x4*)(orow + c) = y;
    }
  }
}

template <int CPT>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* x, const bf16* gain, bf16* out,
                                                      int hidden, float eps) {
  __shared__ float red[4];
  const size_t at = (size_t)blockIdx.x * hidden;
  normalise_row<CPT>(ResidualRow{x + at}, gain, out + at, hidden, eps, red);
}

// Everything a row needs before the first layer, one block per row: cos/sin of
// position * theta^(-2j/d) (angles in double precision), the embedding into the
// residual stream, and its RMSNorm.  In launches of their own the three took
// 2.2 + 2.2 + 2.6 us at 16 rows of 256 columns and 4.8 + 24.5 + 16.3 at 4096
// rows of 4096 (a launch costs about 2 us whatever it does).
template <int CPT>
__global__ __launch_bounds__(256) void row_front_kernel(const TokInfo* toks, const int32_t* tokens,
                                                        const bf16* table, const bf16* gain, float* x,
                                                        bf16* out, int hidden, float eps, int half,
                                                        int head_dim, double theta, float2* cs) {
  __shared__ float red[4];
  const int row = blockIdx.x;
  const size_t at = (size_t)row * hidden;
  normalise_row<CPT>(EmbeddedRow{table + (size_t)tokens[row] * hidden, x + at}, gain, out + at, hidden,
                     eps, red);
  const int j = threadIdx.x;
  if (j < half) {
    const double freq = pow(theta, -2.0 * (double)j / (double)head_dim);
    const double ang = (double)toks[row].pos * freq;
    double sn, cn;
    sincos(ang, &sn, &cn);
    cs[(size_t)row * half + j] = make_float2((float)cn, (float)sn);
  }
}

// Row maximum over the LM-head partials; ties go to the lowest token id.
__global__ __launch_bounds__(256) void argmax_reduce_kernel(const float* part_val,
                                                            const int32_t* part_idx, int parts,
                                                            int32_t* argmax, int32_t* dbg_argmax) {
  // (max, lowest index) is the same whatever order the partials are visited
  // in, so each thread loads eight of them before comparing any: one memory
  // round trip per 2048 partials instead of a dependent load per step.
  constexpr int U = 8;
  __shared__ float sv[4];
  __shared__ int si[4];
  const int row = blockIdx.x;
  const float* pvr = part_val + (size_t)row * parts;
  const int32_t* pir = part_idx + (size_t)row * parts;
  float v = -INFINITY;
  int idx = 0x7fffffff;
  for (int p0 = threadIdx.x; p0 < parts; p0 += 256 * U) {
    float pv[U];
    int pi[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + 256 * u;
      pv[u] = p < parts ? pvr[p] : -INFINITY;
      pi[u] = p < parts ? pir[p] : 0x7fffffff;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (pv[u] > v || (pv[u] == v && pi[u] < idx)) { v = pv[u]; idx = pi[u]; }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const float ov = __shfl_xor(v, m);
    const int oi = __shfl_xor(idx, m);
    if (ov > v || (ov == v && oi < idx)) { v = ov; idx = oi; }
  }
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = v; si[threadIdx.x >> 6] = idx; }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w)
      if (sv[w] > v || (sv[w] == v && si[w] < idx)) { v = sv[w]; idx = si[w]; }
    if (idx == 0x7fffffff) idx = 0;   // every logit NaN: report token 0
    argmax[row] = idx;
    if (dbg_argmax) dbg_argmax[row] = idx;
  }
}

// Greedy tree acceptance, one block per sample, thread i = node i.  A node is
// accepted when on its whole branch every node below the root carries its
// parent's greedy successor, and no proper ancestor is the EOS token (eos = -1:
// none); the deepest accepted node (lowest index on ties) ends the accepted
// branch, and the next token is its greedy successor, or -1 after EOS.  With the
// ancestor sets at hand that is two ballots, a mask test and a maximum (a thread
// that walks its sample's nodes, each a chain of dependent loads, took 9 us at 4
// nodes, 34 at 64 and 59 for 64 samples of 64).
__global__ __launch_bounds__(kMaxTree) void accept_kernel(const SampleInfo* samples,
                                                          const int32_t* tokens, const int32_t* parents,
                                                          const TokInfo* toks, const uint64_t* anc,
                                                          const int32_t* argmax, int eos,
                                                          int32_t* accepted_len, int32_t* next_token,
                                                          int32_t* accepted_nodes) {
  static_assert(kMaxTree == 64 * kAncWords, "one wave per ancestor word");
  __shared__ uint64_t ok[kAncWords], end[kAncWords];
  __shared__ int wave_best[kAncWords];
  const int b = blockIdx.x, i = threadIdx.x, w = i >> 6;
  const SampleInfo s = samples[b];
  const bool live = i < s.ntok;
  const int row = s.tok0 + (live ? i : 0);
  const int tok = tokens[row], depth = toks[row].depth;
  const int parent = live && i > 0 ? parents[row] : 0;
  uint64_t set[kAncWords];
#pragma unroll
  for (int k = 0; k < kAncWords; ++k) set[k] = anc[(size_t)row * kAncWords + k];
  const uint64_t ok_w = __ballot(live && (i == 0 || tok == argmax[s.tok0 + parent]));
  const uint64_t end_w = __ballot(live && tok == eos);
  if ((i & 63) == 0) {
    ok[w] = ok_w;
    end[w] = end_w;
  }
  __syncthreads();
  bool acc = live;
#pragma unroll
  for (int k = 0; k < kAncWords; ++k) {
    const uint64_t above = k == w ? set[k] & ~(1ull << (i & 63)) : set[k];
    acc = acc && (set[k] & ~ok[k]) == 0 && (above & end[k]) == 0;
  }
  int best = acc ? depth * kMaxTree + (kMaxTree - 1 - i) : -1;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) best = max(best, __shfl_xor(best, m));
  if ((i & 63) == 0) wave_best[w] = best;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kAncWords; ++k) best = max(best, wave_best[k]);      // the root is accepted
  const int len = best / kMaxTree, node = kMaxTree - 1 - best % kMaxTree;
  const bool on_branch = live && ((anc[(size_t)(s.tok0 + node) * kAncWords + w] >> (i & 63)) & 1ull);
  int32_t* out = accepted_nodes + (size_t)b * kMaxTree;
  if (on_branch) out[depth] = i;       // the branch has one node per depth 0 .. len
  if (i > len) out[i] = -1;
  if (i == 0) {
    accepted_len[b] = len;
    next_token[b] = tokens[s.tok0 + node] == eos ? -1 : argmax[s.tok0 + node];
  }
}

// Move the accepted branch of one sample, for one layer and a group of K/V heads, to positions
// S_b + 1 .. S_b + accepted_len: row d takes the row of node path[d] > d (rows with path[d] == d
// stay).  Every row written before row d lies below d, and every source of row d or later lies
// above it, so the chunks go in passes of increasing d.  Within a pass a source can be the
// destination of a deeper row, so each pass reads all its chunks into registers, the work-group
// synchronises, and then the pass writes.
template <int HD>
__global__ __launch_bounds__(256) void compact_kernel(const SampleInfo* samples, bf16* kv_pool,
                                                      int n_kv_heads, int heads_per_wg,
                                                      const int32_t* accepted_len,
                                                      const int32_t* accepted_nodes,
                                                      int32_t* new_seq_lens) {
  constexpr int DC = HD / 8;  // 16-byte chunks per row of one head
  constexpr int PER = 8;      // chunks per thread and pass
  const int b = blockIdx.x, layer = blockIdx.y;
  const SampleInfo s = samples[b];
  int acc = accepted_len[b];
  if (acc < 0) acc = 0;
  if (acc > s.ntok - 1) acc = s.ntok - 1;
  if (s.seq_len + acc >= s.cap) acc = s.cap - 1 - s.seq_len;
  if (layer == 0 && blockIdx.z == 0 && threadIdx.x == 0) new_seq_lens[b] = s.seq_len + acc + 1;
  if (acc == 0) return;
  const size_t head_stride = (size_t)s.cap * HD;
  bf16* base = kv_pool + s.kv_base +
               ((size_t)layer * 2 * n_kv_heads + (size_t)blockIdx.z * heads_per_wg) * head_stride;
  const int32_t* nodes = accepted_nodes + (size_t)b * kMaxTree;
  const int per_row = heads_per_wg * DC, total = acc * per_row;
  for (int q0 = 0; q0 < total; q0 += 256 * PER) {
    i32x4 v[PER];
    int64_t dst[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int q = q0 + threadIdx.x + 256 * k;
      dst[k] = -1;
      if (q < total) {
        const int d = 1 + q / per_row, r = q % per_row;
        const int nd = nodes[d];
        if (nd > d && nd < s.ntok && s.seq_len + nd < s.cap) {
          const int64_t col = (int64_t)(r / DC) * head_stride + (r % DC) * 8;
          v[k] = *(const i32x4*)(base + col + (int64_t)(s.seq_len + nd) * HD);
          dst[k] = col + (int64_t)(s.seq_len + d) * HD;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (dst[k] >= 0) *(i32x4*)(base + dst[k]) = v[k];
  }
}

}  // namespace

hipError_t launch_tree_meta(const SampleInfo* samples, int batch, const int32_t* parents,
                            TokInfo* toks, uint64_t* anc, int32_t* dbg_depth, int32_t* dbg_pos,
                            uint64_t* dbg_anc, hipStream_t s) {
  tree_meta_kernel<<<batch, kMaxTree, 0, s>>>(samples, parents, toks, anc, dbg_depth, dbg_pos,
                                               dbg_anc);
  return hipGetLastError();
}

namespace {

// Call `go` with the chunks per thread (an integral_constant) of a row of
// `hidden` columns.
template <class F>
void with_chunks(int hidden, F&& go) {
  switch ((hidden + 1023) / 1024) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3:
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: case 6: case 7:
    case 8: go(std::integral_constant<int, 8>{}); break;
    default: go(std::integral_constant<int, 0>{}); break;
  }
}

}  // namespace

hipError_t launch_row_front(const TokInfo* toks, const int32_t* tokens, const bf16* table,
                            const bf16* gain, float* x, bf16* out, int n, int hidden, float eps,
                            int head_dim, float theta, float2* cs, hipStream_t s) {
  with_chunks(hidden, [&](auto c) {
    row_front_kernel<decltype(c)::value><<<n, 256, 0, s>>>(toks, tokens, table, gain, x, out, hidden, eps,
                                                           head_dim / 2, head_dim, (double)theta, cs);
  });
  return hipGetLastError();
}

hipError_t launch_rmsnorm(const float* x, const bf16* gain, bf16* out, int n, int hidden,
                          float eps, hipStream_t s) {
  with_chunks(hidden, [&](auto c) {
    rmsnorm_kernel<decltype(c)::value><<<n, 256, 0, s>>>(x, gain, out, hidden, eps);
  });
  return hipGetLastError();
}

hipError_t launch_argmax_reduce(const float* part_val, const int32_t* part_idx, int n, int parts,
                                int32_t* argmax, int32_t* dbg_argmax, hipStream_t s) {
  argmax_reduce_kernel<<<n, 256, 0, s>>>(part_val, part_idx, parts, argmax, dbg_argmax);
  return hipGetLastError();
}

hipError_t launch_accept(const SampleInfo* samples, int batch, const int32_t* tokens,
                         const int32_t* parents, const TokInfo* toks, const uint64_t* anc,
                         const int32_t* argmax, int eos, int32_t* accepted_len, int32_t* next_token,
                         int32_t* accepted_nodes, hipStream_t s) {
  accept_kernel<<<batch, kMaxTree, 0, s>>>(samples, tokens, parents, toks, anc, argmax, eos, accepted_len,
                                           next_token, accepted_nodes);
  return hipGetLastError();
}

hipError_t launch_compact(const SampleInfo* samples, int batch, bf16* kv_pool, int n_layers,
                          int n_kv_heads, int head_dim, const int32_t* accepted_len,
                          const int32_t* accepted_nodes, int32_t* new_seq_lens, hipStream_t s) {
  // Head groups split each (sample, layer) only as far as it takes to give the launch about
  // a thousand work-groups: at large batch one work-group moves all K/V heads of a layer.
  const int heads = 2 * n_kv_heads;
  int groups = 1;
  while (groups < heads && (int64_t)batch * n_layers * groups < 1024) {
    ++groups;
    while (heads % groups) ++groups;
  }
  const dim3 grid(batch, n_layers, groups);
  const int hpw = heads / groups;
  if (head_dim == 128)
    compact_kernel<128><<<grid, 256, 0, s>>>(samples, kv_pool, n_kv_heads, hpw, accepted_len,
                                             accepted_nodes, new_seq_lens);
  else if (head_dim == 64)
    compact_kernel<64><<<grid, 256, 0, s>>>(samples, kv_pool, n_kv_heads, hpw, accepted_len,
                                            accepted_nodes, new_seq_lens);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace spec
