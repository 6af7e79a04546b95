// KV transfer buffer for sample migration (RLHFSpec Section 6.2, "Two-stage
// Sample Migration", phases 1 and 3): the K/V of chosen token ranges of
// several samples is copied out of the KV pool into one contiguous buffer, so
// that a migration is a single copy, and parsed back into another pool.
//
// Buffer order (the paper's model -> layer -> sample hierarchy; the LLM is the
// only model here):
//   [layer][K=0,V=1][sample j in call order][kv_head][token t in [begin_j, end_j)][head_dim]
// so every (layer, K/V, sample, head) run of count_j * head_dim values is
// contiguous both in the buffer and in the pool (where one (layer, K/V, head)
// of a sample is [capacity][head_dim]).
//
// One work-group copies one chunk of kChunk 16-byte units of one such run:
// the grid is ordered [layer, K/V][sample][head][chunk], the work-group
// decodes its run once (a binary search over the samples' work-group prefix),
// then streams the chunk with every load of a thread in flight before its
// stores.  The copy is HBM-bound: 2 bytes moved per byte of K/V, each touched
// once, so loads and stores are non-temporal and pass through L2 without
// displacing one another.  Chunks are small (8 KB, two units per thread), which
// measured fastest; presumably a mix of short-lived waves keeps loads and stores
// both in flight, where 16 units per thread are a burst of either.  TB/s moved,
// pack / unpack of 16 samples (8B shape, 32 layers) and of 64 (8 layers, median
// 300 tokens):
//   64 KB chunks, cached           5.1 / 5.1   5.1 / 5.1
//   64 KB, non-temporal (whole pass, pack and unpack)  5.1
//   32 KB, non-temporal (whole pass)                   3.7
//   16 KB, cached                  5.2 / 5.2   5.2 / 5.1
//   16 KB, non-temporal stores     5.4 / 5.3   5.5 / 5.2
//   16 KB, non-temporal            5.8 / 5.6   5.7 / 5.4
//    8 KB, non-temporal            6.2 / 5.9   5.9 / 5.7
//    4 KB, non-temporal            5.9 / 5.9   5.3 / 5.3
#include <algorithm>

#include "common.h"

namespace spec {

namespace {

constexpr int kChunk = 512;                // 16-byte units per work-group (8 KB)
constexpr int kPer = kChunk / 256;         // units per thread
// Work-groups of one launch: HIP holds grid x block, in threads, in 32 bits and
// cuts a larger grid short without an error (16,793,600 work-groups ran 16,384).
// At 8 KB a work-group that is 137 GB, 69 GB when every run ends just past a
// chunk: less than a card can hold, so a larger transfer takes several launches.
constexpr int64_t kMaxGrid = 0xffffffffll / 256;

template <bool TO_BUFFER>
__global__ __launch_bounds__(256) void kv_transfer_kernel(const MigrateInfo* info, int n,
                                                          int64_t first_wg, int64_t wg_per_slab,
                                                          int tok_total, bf16* pool, bf16* buf,
                                                          int n_kv_heads, int head_dim) {
  const int64_t wg = first_wg + blockIdx.x;
  const int lk = (int)(wg / wg_per_slab);            // layer * 2 + (K=0, V=1)
  const int64_t rem = wg % wg_per_slab;
  // Sample whose work-groups cover `rem`: last j with info[j].wg_prefix <= rem.
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (info[mid].wg_prefix <= rem) lo = mid;
    else hi = mid - 1;
  }
  const MigrateInfo m = info[lo];
  const int64_t r2 = rem - m.wg_prefix;
  const int head = (int)(r2 / m.chunks), chunk = (int)(r2 % m.chunks);
  const int dc = head_dim / 8;
  const int64_t units = (int64_t)m.count * dc;       // 16-byte units of this run
  const int64_t u0 = (int64_t)chunk * kChunk;
  bf16* p = pool + m.kv_base + (((int64_t)lk * n_kv_heads + head) * m.cap + m.begin) * head_dim;
  bf16* b = buf + (((int64_t)lk * tok_total + m.tok_prefix) * n_kv_heads + (int64_t)head * m.count) *
                      head_dim;
  const i32x4* src = (const i32x4*)(TO_BUFFER ? p : b);
  i32x4* dst = (i32x4*)(TO_BUFFER ? b : p);
  i32x4 v[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int64_t u = u0 + threadIdx.x + 256 * k;
    if (u < units) v[k] = __builtin_nontemporal_load(src + u);
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int64_t u = u0 + threadIdx.x + 256 * k;
    if (u < units) __builtin_nontemporal_store(v[k], dst + u);
  }
}

}  // namespace

int64_t kv_transfer_chunks(int count, int head_dim) {
  const int64_t units = (int64_t)count * (head_dim / 8);
  return units == 0 ? 0 : (units + kChunk - 1) / kChunk;
}

hipError_t launch_kv_transfer(bool to_buffer, const MigrateInfo* info, int n, int64_t wg_per_slab,
                              int tok_total, bf16* pool, bf16* buf, int n_layers, int n_kv_heads,
                              int head_dim, hipStream_t s) {
  if (wg_per_slab == 0) return hipSuccess;
  const int64_t total = (int64_t)n_layers * 2 * wg_per_slab;
  const auto kernel = to_buffer ? kv_transfer_kernel<true> : kv_transfer_kernel<false>;
  for (int64_t first = 0; first < total; first += kMaxGrid) {
    const int64_t grid = std::min(kMaxGrid, total - first);
    kernel<<<(unsigned)grid, 256, 0, s>>>(info, n, first, wg_per_slab, tok_total, pool, buf, n_kv_heads,
                                          head_dim);
    if (const hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

}  // namespace spec
