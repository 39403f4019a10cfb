// Splice of a compiled KV block into a paged KV cache (Sec. VI-A; transposed V per Sec. VI-B).
//
// Pure data movement, bit-exact.  Block rows [l][j][h][:] are contiguous; cache rows
// [l][page][h][slot][:] are contiguous, so the row-major kernel streams 16-byte chunks in the
// block's own order (coalesced reads) and writes whole rows (256 B for bf16, head_dim 128),
// both with non-temporal accesses (config 3, 48 layers, steady state: 70.6 -> 64.6 us).
// The transposed-V kernel transposes 16-byte x 16-byte blocks in registers: whole rows are read, and
// every feature row of the cache is written a page (32 or 64 bytes) at a time.
#include "device_common.h"
#include "launch.h"

#include <algorithm>

namespace nexus {

constexpr int kSpliceItemsPerThread = 1;

// Row-major splice of K and V (blockIdx.z: 0 = K, 1 = V; z = 1 is skipped for a transposed V).
// Work item = one 16-byte chunk; a layer's items are ordered (token j, head h, chunk c).
__global__ __launch_bounds__(256) void splice_rows_kernel(
    const u32x4 *__restrict__ bk, const u32x4 *__restrict__ bv, u32x4 *__restrict__ ck,
    u32x4 *__restrict__ cv, const int32_t *__restrict__ map, int64_t offset,
    uint32_t items_per_layer, uint32_t chunks_per_row, uint32_t chunk_shift, FastDiv div_heads,
    uint32_t n_heads, uint32_t n_phys_pages, uint32_t n_tokens) {
  const uint32_t layer = blockIdx.y;
  const u32x4 *src = blockIdx.z == 0 ? bk : bv;
  u32x4 *dst = blockIdx.z == 0 ? ck : cv;
  const uint64_t src_layer = (uint64_t)layer * items_per_layer;
  const uint64_t dst_layer = (uint64_t)layer * n_phys_pages * n_heads * kPage * chunks_per_row;
  // items per thread and loop pass: one item per thread, many workgroups (config 3, 48 layers:
  // 66.0 us against 69.2 us with four items per thread and a quarter of the workgroups)
  constexpr int kUnroll = kSpliceItemsPerThread;
  const uint32_t stride = gridDim.x * blockDim.x;
  uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x;
  for (; idx < items_per_layer; idx += kUnroll * stride) {
    u32x4 v[kUnroll];
    uint64_t daddr[kUnroll];
    bool ok[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const uint32_t i = idx + u * stride;
      ok[u] = i < items_per_layer;
      const uint32_t ii = ok[u] ? i : idx;
      const uint32_t row = ii >> chunk_shift;          // j * H + h
      const uint32_t c = ii & (chunks_per_row - 1);
      const uint32_t j = fdiv(row, div_heads);
      const uint32_t h = row - j * n_heads;
      const int64_t t = offset + j;
      const uint32_t page = (uint32_t)map[t >> kPageShift];
      const uint32_t slot = (uint32_t)(t & (kPage - 1));
      daddr[u] = dst_layer + (((uint64_t)page * n_heads + h) * kPage + slot) * chunks_per_row + c;
      v[u] = ld_stream(src + src_layer + ii);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (ok[u]) st_stream(v[u], dst + daddr[u]);
  }
  (void)n_tokens;
}

// Transposed-V splice.  A thread takes an E x E block (E = 16 bytes of elements: 8 bf16, 4 f32): E
// tokens of one logical page, one 16-byte chunk of features.  It loads the chunk from E block rows,
// all in flight together, and stores E tokens to each of the E feature rows; the 16 / E blocks of a
// page sit in adjacent lanes, so a page is one 32- or 64-byte piece of a feature row.  Only tokens
// inside [offset, offset + n_tokens) are written.
// The pieces bound it: where logical pages are neighbours in memory, pieces of several pages make up
// a cache line, so all pages of a (layer, head) go to one XCD (ids 8 apart), whose L2 joins them.
// The rows are read past the caches, which keeps the lines that wait for their other pieces in them.
// Shuffled pages, through an LDS tile with a head's pages over all XCDs, then so: 26 layers x 512 tokens x 8
// heads of 256 bf16 cold 76 -> 55 us (the whole splice 73 -> 61, with cached reads 69); an append
// whose tokens were just written 65 -> 50; one block spliced into the same pages over and over, which
// cached reads would find in the last-level cache, 51 -> 59 (46).
template <typename T>
__global__ __launch_bounds__(256) void splice_vt_kernel(
    const T *__restrict__ bv, T *__restrict__ cvt, const int32_t *__restrict__ map,
    int64_t offset, int32_t n_tokens, int32_t n_heads, int32_t head_dim, uint32_t chunk_shift,
    int32_t n_phys_pages, int32_t n_pages, uint32_t n_groups, uint32_t first_group) {
  constexpr int E = 16 / (int)sizeof(T);
  constexpr int PB = kPage / E;                       // blocks per page and chunk
  const uint32_t group = first_group + 8 * blockIdx.y + (blockIdx.x & 7);   // layer * n_heads + head
  if (group >= n_groups) return;                      // padding of the grid
  const uint32_t item = (blockIdx.x >> 3) * 256 + threadIdx.x;
  const int g = item % PB;
  const int c = (item / PB) & ((1u << chunk_shift) - 1);
  const int p = (int)(item / PB >> chunk_shift);
  if (p >= n_pages) return;
  const int64_t page0 = offset >> kPageShift;
  const int64_t t0 = (page0 + p) * kPage + g * E, t_end = offset + n_tokens;
  if (t0 + E <= offset || t0 >= t_end) return;        // no block token here
  const uint32_t layer = group / (uint32_t)n_heads, h = group - layer * n_heads;
  const int64_t phys = (uint32_t)map[page0 + p];
  const T *src = bv + ((int64_t)layer * n_tokens * n_heads + h) * head_dim + c * E;
  const int64_t row = (int64_t)n_heads * head_dim;
  u32x4 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int64_t t = t0 + e < offset ? offset : t0 + e < t_end ? t0 + e : t_end - 1;
    v[e] = ld_stream(reinterpret_cast<const u32x4 *>(src + (t - offset) * row));
  }
  const int64_t n_cols = (int64_t)n_phys_pages * kPage;
  T *dst = cvt + ((int64_t)group * head_dim + c * E) * n_cols + phys * kPage + g * E;
  const bool whole = t0 >= offset && t0 + E <= t_end;
#pragma unroll
  for (int d = 0; d < E; ++d) {
    u32x4 w;
    if constexpr (sizeof(T) == 2) {
      const uint32_t sel = (d & 1) ? 0x07060302u : 0x05040100u;   // high or low halves
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = __builtin_amdgcn_perm(v[2 * i + 1][d >> 1], v[2 * i][d >> 1], sel);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = v[i][d];
    }
    if (whole) {
      *reinterpret_cast<u32x4 *>(dst + d * n_cols) = w;
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const T x = sizeof(T) == 2 ? (T)(w[e * sizeof(T) / 4] >> (16 * (e & 1))) : (T)w[e & 3];
        if (t0 + e >= offset && t0 + e < t_end) dst[d * n_cols + e] = x;
      }
    }
  }
}

hipError_t launch_splice(const SpliceLaunch &p, hipStream_t stream) {
  const uint32_t esize = p.dtype_bytes;
  const uint32_t chunks_per_row = (uint32_t)p.head_dim * esize / 16;
  uint32_t shift = 0;
  while ((1u << shift) < chunks_per_row) ++shift;
  const uint64_t items = (uint64_t)p.n_tokens * p.n_heads * chunks_per_row;
  const int n_kv = p.v_transposed ? 1 : 2;
  if (!p.v_only) {
    const uint32_t threads = 256;
    uint64_t want = (items + threads * kSpliceItemsPerThread - 1) / (threads * kSpliceItemsPerThread);
    const uint32_t blocks = (uint32_t)(want < 1 ? 1 : (want > 65535 ? 65535 : want));
    dim3 grid(blocks, p.n_layers, n_kv);
    hipLaunchKernelGGL(splice_rows_kernel, grid, dim3(threads), 0, stream,
                       (const u32x4 *)p.block_k, (const u32x4 *)p.block_v, (u32x4 *)p.cache_k,
                       (u32x4 *)p.cache_v, p.map, p.offset, (uint32_t)items, chunks_per_row, shift,
                       make_fastdiv(p.n_heads), (uint32_t)p.n_heads, (uint32_t)p.n_phys_pages,
                       (uint32_t)p.n_tokens);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (p.v_transposed) {
    // the entry points take transposed rows of up to 512 bytes (head_dim 256 in bf16, 128 in f32)
    if (p.head_dim * esize > 512) return hipErrorInvalidValue;
    const int32_t n_pages = (int32_t)(((p.offset + p.n_tokens - 1) >> kPageShift) -
                                      (p.offset >> kPageShift) + 1);
    const uint32_t n_groups = (uint32_t)p.n_layers * (uint32_t)p.n_heads;
    const uint64_t blocks = (uint64_t)n_pages * chunks_per_row * (kPage * esize / 16);
    const uint32_t wpg = (uint32_t)((blocks + 255) / 256);
    // grid y: 8 groups each (at most 65535 of them to a launch), x: their workgroups in turn
    for (uint32_t g0 = 0; g0 < n_groups; g0 += 8 * 65535u) {
      const dim3 grid(8 * wpg, std::min<uint32_t>((n_groups - g0 + 7) / 8, 65535u));
#define NEXUS_SPLICE_VT(T)                                                                          \
  hipLaunchKernelGGL(splice_vt_kernel<T>, grid, dim3(256), 0, stream, (const T *)p.block_v,         \
                     (T *)p.cache_v, p.map, p.offset, p.n_tokens, p.n_heads, p.head_dim, shift,     \
                     p.n_phys_pages, n_pages, n_groups, g0)
      if (esize == 2) NEXUS_SPLICE_VT(uint16_t);
      else NEXUS_SPLICE_VT(uint32_t);
#undef NEXUS_SPLICE_VT
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace nexus
