// Semantic Lookaside Buffer scan on MI355X (Sec. V-A): INT8 tool embeddings scanned with integer
// dot products against INT8 query embeddings, the best tools per query kept, and the margin gate
// (auto-route when the top-two score margin exceeds tau, else escalate).
//
// Score of tool t for query q: (float(dot_int32(T_t, Q_q)) * s_t) * s_q in fp32, each product
// rounded to nearest-even; the integer dot is exact and, with |dot| <= 127^2 * 1024 < 2^24,
// exactly representable in fp32.
//
// The scan kernels compute S^T = T.Q^T on v_mfma_i32_16x16x64_i8 (tool rows straight from
// global memory into the A-operand registers, the query block staged in LDS as the B operands),
// loading ahead while they compute.  Lane l then holds tools 4 (l / 16) .. +3 of a 16-tool tile
// for query column l % 16.  A candidate is one 64-bit key that carries both orders (higher score
// first, lower index first among equal scores), so the best are found by comparing keys alone.
//
// * Up to 16 queries (the single-query lookup of a user turn), and many over a registry of
//   one range: one 16-query block per workgroup column; the waves take the range's 16-tool tiles
//   in turn, each tile one MFMA chain, and fold the scores into each lane's own sorted list of the
//   best KT.  A column's 4 lane lists are merged by lane exchanges and the 4 waves' lists through
//   LDS.  With one range the result is final (top-k, margin, gate); otherwise each range's best
//   go to the workspace and a second kernel merges them.  HBM-bound for one query.
// * Thousands of queries over a small registry (slb_block_kernel): the same lists, for 64 queries a workgroup.
// * More queries: two passes without any list in the first (slb_max_kernel, slb_select_kernel).
//   The first writes the best score of every 16-tool tile for every query; the second takes the
//   KT best tiles of a query, which hold its KT best tools (a tool of any other tile has KT tools
//   ranking above it, one in each of those tiles: equal scores go to the lower tile as to the lower
//   index), scores their KT x 16 tools again and ranks them.
#include "device_common.h"
#include "launch_slb.h"

#include <algorithm>

namespace nexus {

namespace {

typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr int kTop = 8;          // candidates kept per (lane, query) and per range
constexpr int kWaves = 4;
constexpr int kSubBlocks = 4;    // 16-query sub-blocks per workgroup (64 queries)
// LDS row padding of the staged query block: dim is a multiple of 64 bytes, so unpadded rows
// start on the same bank and the 16 rows an MFMA B operand reads would all hit the same 4 banks
constexpr int kQPad = 16;

// A candidate (score, tool index) is one 64-bit key whose unsigned order is the ranking order:
// the fp32 score mapped to an order-preserving 32-bit pattern in the high half, the complement
// of the index in the low half (so the lower index wins between equal scores); 0 = no tool.
__device__ __forceinline__ uint64_t cand_key(float score, int idx) {
  const uint32_t u = __float_as_uint(score);
  const uint32_t ord = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ((uint64_t)ord << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)idx);
}
__device__ __forceinline__ int cand_idx(uint64_t k) {
  return k == 0 ? -1 : (int)(0xFFFFFFFFu - (uint32_t)k);
}
__device__ __forceinline__ float cand_score(uint64_t k) {
  if (k == 0) return -INFINITY;
  const uint32_t ord = (uint32_t)(k >> 32);
  return __uint_as_float((ord & 0x80000000u) ? (ord & 0x7FFFFFFFu) : ~ord);
}

// Insert x into the descending list b: a max/min pass carries x down to its place and drops the
// smallest.  Skipped by the whole wave when no lane's x beats its list's last entry.
template <int KT>
__device__ __forceinline__ void insert(uint64_t (&b)[KT], uint64_t x) {
  if (!__builtin_amdgcn_ballot_w64(x > b[KT - 1])) return;
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    const bool gt = x > b[j];
    const uint64_t hi = gt ? x : b[j];
    x = gt ? b[j] : x;
    b[j] = hi;
  }
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int off) {
  const uint32_t lo = __shfl_xor((uint32_t)v, off);
  const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), off);
  return ((uint64_t)hi << 32) | lo;
}

// The best KT of n candidate keys, selected by one wave: every lane sorts its
// share, then KT rounds take the wave-wide largest head (keys are distinct, so exactly one lane
// advances).
template <int KT>
__device__ __forceinline__ void wave_select(const uint64_t *c, int n, int lane,
                                            uint64_t (&out)[KT]) {
  uint64_t b[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) b[j] = 0;
  for (int i = lane; i < n; i += 64) insert<KT>(b, c[i]);
  int head = 0;
#pragma unroll
  for (int r = 0; r < KT; ++r) {
    uint64_t h = 0;
#pragma unroll
    for (int j = 0; j < KT; ++j) h = j == head ? b[j] : h;
    uint64_t w = h;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const uint64_t o = shfl_xor_u64(w, off);
      w = o > w ? o : w;
    }
    out[r] = w;
    if (w != 0 && h == w) ++head;
  }
}

struct SlbArgs {
  const int8_t *tools;
  const float *tool_scale;
  const int8_t *queries;
  const float *query_scale;
  int32_t n_tools, n_queries, dim, k;
  int32_t n_ranges, range_tools;     // tools per range (a multiple of 64)
  float tau;
  int32_t *top_idx;
  float *top_score;
  float *margin;
  int32_t *route;
  uint64_t *part;                     // [n_queries][n_ranges][KT] candidate keys
  uint32_t *tile_max;                 // batches: [n_queries][tile_ld] best score of each tile
  int32_t tile_ld, n_qblocks;         // 16-tool tiles of whole 64-tool blocks; 64-query blocks
};

// Final outputs of one query from its sorted best keys (lane 0 writes).
template <int KT>
__device__ __forceinline__ void write_final(const SlbArgs &a, int q, const uint64_t (&b)[KT],
                                            int lane) {
  if (lane != 0) return;
#pragma unroll
  for (int j = 0; j < KT; ++j)
    if (j < a.k) {
      a.top_idx[(size_t)q * a.k + j] = cand_idx(b[j]);
      a.top_score[(size_t)q * a.k + j] = cand_score(b[j]);
    }
  // fewer than two tools: nothing to confuse the best one with
  const float m = b[1] == 0 ? INFINITY : cand_score(b[0]) - cand_score(b[1]);
  a.margin[q] = m;
  a.route[q] = m > a.tau ? 1 : 0;
}

// A lower bound of the KT-th best key of a query column whose candidates are spread over 4 lane
// lists (lanes l, l ^ 16, l ^ 32, l ^ 48), each sorted descending: the largest of the lanes'
// KT-th entries, and the smallest of the lanes' (KT/4)-th entries (every lane then holds at least
// KT/4 keys at or above it, KT in all).  The second is the tight one while the lists are short
// of candidates of their own: after the first tile or block it sits near the column's KT-th best.
template <int KT>
__device__ __forceinline__ uint64_t column_floor(const uint64_t (&b)[KT]) {
  uint64_t f = b[KT - 1];
  uint64_t g = b[KT >= 4 ? KT / 4 - 1 : 0];
  uint64_t o = shfl_xor_u64(f, 16);
  f = o > f ? o : f;
  o = shfl_xor_u64(f, 32);
  f = o > f ? o : f;
  o = shfl_xor_u64(g, 16);
  g = o < g ? o : g;
  o = shfl_xor_u64(g, 32);
  g = o < g ? o : g;
  return f > g ? f : g;
}

// Merge the partner lane's sorted list into this lane's (both lanes end with the best KT of the
// union, the same list).
template <int KT>
__device__ __forceinline__ void merge_lanes(uint64_t (&b)[KT], int off) {
  uint64_t o[KT];
#pragma unroll
  for (int j = 0; j < KT; ++j) o[j] = shfl_xor_u64(b[j], off);
#pragma unroll
  for (int j = 0; j < KT; ++j) {
    uint64_t x = o[j];
#pragma unroll
    for (int m = 0; m < KT; ++m) {
      const bool gt = x > b[m];
      const uint64_t hi = gt ? x : b[m];
      x = gt ? b[m] : x;
      b[m] = hi;
    }
  }
}

// Small batches (the single-query lookup of a user turn): workgroup = range; registries of one range:
// workgroup = 16-query block.
// MAXS: 64-byte steps of dim at most (dim <= 64 MAXS); KT: candidates kept, >= max(k, 2).  The
// query block sits in LDS; wave w takes the range's 16-tool tiles w, w + 4, ..., loading each
// tile's rows straight into the A-operand registers (the next tile in flight) and running one
// MFMA chain per tile; the 4 waves' lists of a query meet in LDS.
template <int MAXS, int KT>
__global__ __launch_bounds__(256) void slb_scan_kernel(SlbArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  int8_t *qs = reinterpret_cast<int8_t *>(smem);                       // [16][dim + kQPad]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  const int range = blockIdx.y;
  const int q0 = 16 * blockIdx.x, n_q = min(16, a.n_queries - q0);
  const int t_begin = range * a.range_tools;
  const int t_end = min(t_begin + a.range_tools, a.n_tools);
  const int dim = a.dim, steps = dim / 64, ld = dim + kQPad;

  // stage the query block (rows past n_queries are zero)
  for (int c = tid; c < 16 * (dim / 16); c += 256) {
    const int r = c / (dim / 16), off = (c - r * (dim / 16)) * 16;
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (r < n_q) v = *reinterpret_cast<const u32x4 *>(a.queries + (size_t)(q0 + r) * dim + off);
    *reinterpret_cast<u32x4 *>(qs + r * ld + off) = v;
  }
  const float sq = qn < n_q ? a.query_scale[q0 + qn] : 0.f;
  __syncthreads();

  uint64_t best[KT];
  uint64_t floor_key = 0;   // a lower bound of the KT-th best key of this lane's query column
#pragma unroll
  for (int j = 0; j < KT; ++j) best[j] = 0;

  struct Tile {
    i32x4 a[MAXS];
    float st[4];
  };
  // Every call issues the same loads (rows and steps past the end re-read valid ones), so the
  // wait before a tile's use leaves the next tile's loads in flight.
  auto load_tile = [&](int t0, Tile &tl) {
    const int8_t *trow = a.tools + (size_t)min(t0 + qn, a.n_tools - 1) * dim + 16 * grp;
#pragma unroll
    for (int st = 0; st < MAXS; ++st)
      tl.a[st] = *reinterpret_cast<const i32x4 *>(trow + 64 * min(st, steps - 1));
#pragma unroll
    for (int i = 0; i < 4; ++i) tl.st[i] = a.tool_scale[min(t0 + 4 * grp + i, a.n_tools - 1)];
  };
  auto compute_tile = [&](int t0, const Tile &tl) {
    i32x4 acc = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int st = 0; st < MAXS; ++st) {
      if (st < steps) {
        const i32x4 bv = *reinterpret_cast<const i32x4 *>(qs + qn * ld + 64 * st + 16 * grp);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(tl.a[st], bv, acc, 0, 0, 0);
      }
    }
    // lane: tools t0 + 4 grp + i for query column qn.  A candidate that does not beat the
    // column's floor (at most the column's KT-th best) cannot be among its best KT and is
    // dropped.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + 4 * grp + i;
      const float score = ((float)acc[i] * tl.st[i]) * sq;
      const uint64_t key = t < t_end ? cand_key(score, t) : 0;
      insert<KT>(best, key > floor_key ? key : 0);
    }
    floor_key = column_floor<KT>(best);
  };

  // this wave's 16-tool tiles: t_begin + 16 (wave + 4 j)
  {
    const int stride = 16 * kWaves;
    Tile b0, b1;
    int t0 = t_begin + 16 * wave;
    if (t0 < t_end) {
      load_tile(t0, b0);
      for (;;) {
        load_tile(t0 + stride, b1);
        compute_tile(t0, b0);
        t0 += stride;
        if (t0 >= t_end) break;
        load_tile(t0 + stride, b0);
        compute_tile(t0, b1);
        t0 += stride;
        if (t0 >= t_end) break;
      }
    }
  }

  // each column's 4 lists inside the wave, then the other waves' lists through LDS
  merge_lanes<KT>(best, 16);
  merge_lanes<KT>(best, 32);
  __syncthreads();                                                     // query block no longer read
  uint64_t *cl = reinterpret_cast<uint64_t *>(smem);                   // [wave][16][KT]
  if (wave > 0 && grp == 0)
#pragma unroll
    for (int j = 0; j < KT; ++j) cl[(wave * 16 + qn) * KT + j] = best[j];
  __syncthreads();
  if (wave > 0 || grp != 0 || qn >= n_q) return;
  const int q = q0 + qn;
  for (int w = 1; w < kWaves; ++w)
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      uint64_t x = cl[(w * 16 + qn) * KT + j];
#pragma unroll
      for (int m = 0; m < KT; ++m) {
        const bool gt = x > best[m];
        const uint64_t hi = gt ? x : best[m];
        x = gt ? best[m] : x;
        best[m] = hi;
      }
    }
  if (a.n_ranges == 1) {
#pragma unroll
    for (int j = 0; j < KT; ++j)
      if (j < a.k) {
        a.top_idx[(size_t)q * a.k + j] = cand_idx(best[j]);
        a.top_score[(size_t)q * a.k + j] = cand_score(best[j]);
      }
    const float m = best[1] == 0 ? INFINITY : cand_score(best[0]) - cand_score(best[1]);
    a.margin[q] = m;
    a.route[q] = m > a.tau ? 1 : 0;
  } else {
    const size_t o = ((size_t)q * a.n_ranges + range) * KT;
#pragma unroll
    for (int j = 0; j < KT; ++j) a.part[o + j] = best[j];
  }
}

// ---- large batches over small registries: workgroup = 64 queries x one range, its 4 waves take 64-tool
// blocks in turn with 16 MFMA chains each, as slb_max_kernel does, and keep the best KT of every column
// in lane lists.  Most of its time is list upkeep (a wave inserts nearly every score of its first blocks),
// which does not grow with the queries while the chip has room: 300 tools x 64 .. 8192 queries 30 .. 36 us.
template <int KT>
__global__ __launch_bounds__(256, 2) void slb_block_kernel(SlbArgs a) {
  constexpr int QB = 64, NT = 4, NSB = 4, CS = 2;   // queries, tool tiles, sub-blocks, steps
  extern __shared__ __align__(16) unsigned char smem[];
  const int dim = a.dim, steps = dim / 64, ld = dim + kQPad;
  int8_t *qs = reinterpret_cast<int8_t *>(smem);                         // [QB][ld]
  float *tsc = reinterpret_cast<float *>(smem + (size_t)QB * ld);        // [range_tools]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  const int q0 = blockIdx.y * QB;
  const int range = blockIdx.x;
  const int t_begin = range * a.range_tools;
  const int t_end = min(t_begin + a.range_tools, a.n_tools);

  for (int c = tid; c < QB * (dim / 16); c += 256) {
    const int r = c / (dim / 16), off = (c - r * (dim / 16)) * 16;
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (q0 + r < a.n_queries)
      v = *reinterpret_cast<const u32x4 *>(a.queries + (size_t)(q0 + r) * dim + off);
    *reinterpret_cast<u32x4 *>(qs + r * ld + off) = v;
  }
  for (int i = tid; i < t_end - t_begin; i += 256) tsc[i] = a.tool_scale[t_begin + i];
  float sq[NSB];
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    const int q = q0 + 16 * sb + qn;
    sq[sb] = q < a.n_queries ? a.query_scale[q] : 0.f;
  }
  __syncthreads();

  uint64_t best[NSB][KT];
  uint64_t floor_key[NSB];
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    floor_key[sb] = 0;
#pragma unroll
    for (int j = 0; j < KT; ++j) best[sb][j] = 0;
  }

  // this wave's blocks: wave, wave + 4, ... of the range's 64-tool blocks; each is n_chunks
  // chunks of CS steps, walked as one sequence u = block * n_chunks + chunk
  const int n_blocks = (t_end - t_begin + 63) / 64;
  const int my_blocks = n_blocks > wave ? (n_blocks - wave + kWaves - 1) / kWaves : 0;
  const int n_chunks = (steps + CS - 1) / CS;
  const int total = my_blocks * n_chunks;
  struct Chunk {
    i32x4 a[NT][CS];
  };
  // Every call issues the same loads (past the sequence's end it re-reads the last chunk; rows
  // and steps past the registry's end re-read valid ones), so the wait before a chunk's use
  // leaves the next chunk's loads in flight.
  auto load_chunk = [&](int u, Chunk &ch) {
    const int uu = min(u, total - 1);
    const int j = uu / n_chunks, c = uu - j * n_chunks;
    const int t0 = t_begin + 64 * (wave + kWaves * j);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int8_t *trow = a.tools + (size_t)min(t0 + 16 * i + qn, a.n_tools - 1) * dim + 16 * grp;
#pragma unroll
      for (int s2 = 0; s2 < CS; ++s2)
        ch.a[i][s2] = *reinterpret_cast<const i32x4 *>(trow + 64 * min(c * CS + s2, steps - 1));
    }
  };
  i32x4 acc[NT][NSB];
  auto step = [&](int u, const Chunk &ch) {
    const int j = u / n_chunks, c = u - j * n_chunks;
    if (c == 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) acc[i][sb] = i32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int s2 = 0; s2 < CS; ++s2) {
      const int st = c * CS + s2;
      if (st < steps) {
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) {
          const i32x4 bv =
              *reinterpret_cast<const i32x4 *>(qs + (16 * sb + qn) * ld + 64 * st + 16 * grp);
#pragma unroll
          for (int i = 0; i < NT; ++i)
            acc[i][sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ch.a[i][s2], bv, acc[i][sb], 0, 0, 0);
        }
      }
    }
    if (c != n_chunks - 1) return;
    // the candidate pass runs at a raised wave priority, so that its list upkeep interleaves
    // with the other wave's MFMA chains (about 4% faster at 65536 tools x 256 queries)
    __builtin_amdgcn_s_setprio(2);
    // the block's 64 x 64 scores: a candidate that does not beat its column's floor (at most
    // the column's KT-th best) cannot be among the column's best KT and is dropped
    const int tb = 64 * (wave + kWaves * j);                   // block start within the range
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const f32x4 sc = *reinterpret_cast<const f32x4 *>(tsc + tb + 16 * i + 4 * grp);
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int t = t_begin + tb + 16 * i + 4 * grp + r;
          const float score = ((float)acc[i][sb][r] * sc[r]) * sq[sb];
          const uint64_t key = t < t_end ? cand_key(score, t) : 0;
          insert<KT>(best[sb], key > floor_key[sb] ? key : 0);
        }
      }
    }
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) floor_key[sb] = column_floor<KT>(best[sb]);
    __builtin_amdgcn_s_setprio(0);
  };
  if (total > 0) {
    Chunk b0, b1;
    int u = 0;
    load_chunk(0, b0);
    for (;;) {
      load_chunk(u + 1, b1);
      step(u, b0);
      if (++u >= total) break;
      load_chunk(u + 1, b0);
      step(u, b1);
      if (++u >= total) break;
    }
  }

  // each column's 4 lists inside the wave, then the 4 waves' lists through LDS
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    merge_lanes<KT>(best[sb], 16);
    merge_lanes<KT>(best[sb], 32);
  }
  __syncthreads();                                        // query block and scales no longer read
  uint64_t *cl = reinterpret_cast<uint64_t *>(smem);      // [wave][NSB][16][KT]
  if (wave > 0 && grp == 0)
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
      for (int j = 0; j < KT; ++j) cl[((wave * NSB + sb) * 16 + qn) * KT + j] = best[sb][j];
  __syncthreads();
  if (wave > 0 || grp != 0) return;
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    const int q = q0 + 16 * sb + qn;
    if (q >= a.n_queries) continue;
    for (int w = 1; w < kWaves; ++w)
#pragma unroll
      for (int j = 0; j < KT; ++j) {
        uint64_t x = cl[((w * NSB + sb) * 16 + qn) * KT + j];
#pragma unroll
        for (int m = 0; m < KT; ++m) {
          const bool gt = x > best[sb][m];
          const uint64_t hi = gt ? x : best[sb][m];
          x = gt ? best[sb][m] : x;
          best[sb][m] = hi;
        }
      }
    if (a.n_ranges == 1) {
#pragma unroll
      for (int j = 0; j < KT; ++j)
        if (j < a.k) {
          a.top_idx[(size_t)q * a.k + j] = cand_idx(best[sb][j]);
          a.top_score[(size_t)q * a.k + j] = cand_score(best[sb][j]);
        }
      const float m =
          best[sb][1] == 0 ? INFINITY : cand_score(best[sb][0]) - cand_score(best[sb][1]);
      a.margin[q] = m;
      a.route[q] = m > a.tau ? 1 : 0;
    } else {
      const size_t o = ((size_t)q * a.n_ranges + range) * KT;
#pragma unroll
      for (int j = 0; j < KT; ++j) a.part[o + j] = best[sb][j];
    }
  }
}

// ---- batches: pass 1.  Workgroup = 64 queries x one range of tools; its 4 waves take 64-tool blocks
// of the range in turn.  For one block a wave keeps 16 MFMA chains (4 tool tiles x 4 query sub-blocks)
// and walks the dimension two 64-byte steps at a time, holding those steps of its 64 tool rows in
// registers (the next two in flight), so every B operand read from LDS feeds four MFMAs.  Lane
// (qn, grp) loads, for tool tile i of a block, bytes 64 st + 16 grp of tool row 16 i + qn (the A
// operand) and reads bytes 64 st + 16 grp of query row 16 sb + qn from LDS (the B operand); its
// accumulator holds the scores of tools 16 i + 4 grp + r (r = 0..3) for query column 16 sb + qn.
// The best score of each tile (its ordered pattern; 0 for a tile past the registry) goes to
// part[query][tile].  Keeping a sorted list per lane here instead, a wave inserts nearly every
// score it meets, because it meets few tools: 65536 tools x 256 queries of dim 768, k 8, whole
// call: 125 us, this way 46.7 (this pass 33, the second 14).
// Its time grows with dim x queries at about a fifth of the int8 MFMA rate; two more chunks in flight, 8
// waves a workgroup and an unbranched loop changed nothing (34.5, 35.8, 33.8).
__device__ __forceinline__ uint32_t score_order(float score) {
  const uint32_t u = __float_as_uint(score);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ uint32_t umax(uint32_t x, uint32_t y) { return x > y ? x : y; }

__global__ __launch_bounds__(256, 2) void slb_max_kernel(SlbArgs a) {
  constexpr int QB = 64, NT = 4, NSB = 4, CS = 2;   // queries, tool tiles, sub-blocks, steps
  extern __shared__ __align__(16) unsigned char smem[];
  const int dim = a.dim, steps = dim / 64, ld = dim + kQPad;
  int8_t *qs = reinterpret_cast<int8_t *>(smem);                         // [QB][ld]
  float *tsc = reinterpret_cast<float *>(smem + (size_t)QB * ld);        // [range_tools]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  // (range, query block) in that order are cut into 8 equal runs, one to an XCD (ids 8 apart): an XCD's L2
  // then holds the tools of its own ranges, and all XCDs work however few the ranges are
  const int n_items = a.n_ranges * a.n_qblocks;
  const int item = (blockIdx.x & 7) * ((n_items + 7) / 8) + (blockIdx.x >> 3);
  if (item >= n_items || (int)(blockIdx.x >> 3) >= (n_items + 7) / 8) return;   // padding of the grid
  const int range = item / a.n_qblocks;
  const int q0 = (item - range * a.n_qblocks) * QB;
  const int t_begin = range * a.range_tools;
  const int t_end = t_begin + min(a.range_tools, a.n_tools - t_begin);

  // this wave's blocks: wave, wave + 4, ... of the range's 64-tool blocks; each is n_chunks
  // chunks of CS steps, walked as one sequence u = block * n_chunks + chunk
  const int n_blocks = (t_end - t_begin + 63) / 64;
  const int my_blocks = n_blocks > wave ? (n_blocks - wave + kWaves - 1) / kWaves : 0;
  const int n_chunks = (steps + CS - 1) / CS;
  const int total = my_blocks * n_chunks;
  struct Chunk {
    i32x4 a[NT][CS];
  };
  // Every call issues the same loads (past the sequence's end it re-reads the last chunk; rows
  // and steps past the registry's end re-read valid ones), so the wait before a chunk's use
  // leaves the next chunk's loads in flight.
  auto load_chunk = [&](int u, Chunk &ch) {
    const int uu = min(u, total - 1);
    const int j = uu / n_chunks, c = uu - j * n_chunks;
    const int t0 = t_begin + 64 * (wave + kWaves * j);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int8_t *trow = a.tools + (size_t)min(t0 + 16 * i + qn, a.n_tools - 1) * dim + 16 * grp;
#pragma unroll
      for (int s2 = 0; s2 < CS; ++s2)
        ch.a[i][s2] = *reinterpret_cast<const i32x4 *>(trow + 64 * min(c * CS + s2, steps - 1));
    }
  };
  Chunk b0, b1;
  if (total > 0) load_chunk(0, b0);

  // stage the query block: thread tid takes row tid / 4, 16-byte pieces tid % 4, + 4, .. (rows past
  // the batch are zero); kStageSteps loads at a time in flight
  {
    constexpr int kStageSteps = 4;
    const int r = tid >> 2, q = q0 + r;
    const int8_t *row = a.queries + (size_t)min(q, a.n_queries - 1) * dim + 16 * (tid & 3);
    for (int s0 = 0; s0 < steps; s0 += kStageSteps) {
      u32x4 v[kStageSteps];
#pragma unroll
      for (int e = 0; e < kStageSteps; ++e)
        v[e] = *reinterpret_cast<const u32x4 *>(row + 64 * min(s0 + e, steps - 1));
#pragma unroll
      for (int e = 0; e < kStageSteps; ++e)
        if (s0 + e < steps)
          *reinterpret_cast<u32x4 *>(qs + r * ld + 64 * (s0 + e) + 16 * (tid & 3)) =
              q < a.n_queries ? v[e] : u32x4{0u, 0u, 0u, 0u};
    }
  }
  for (int i = tid; i < a.range_tools; i += 256)
    tsc[i] = t_begin + i < t_end ? a.tool_scale[t_begin + i] : 0.f;
  float sq[NSB];
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
    const int q = q0 + 16 * sb + qn;
    sq[sb] = q < a.n_queries ? a.query_scale[q] : 0.f;
  }
  __syncthreads();

  i32x4 acc[NT][NSB];
  auto step = [&](int u, const Chunk &ch) {
    const int j = u / n_chunks, c = u - j * n_chunks;
    if (c == 0) {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) acc[i][sb] = i32x4{0, 0, 0, 0};
    }
#pragma unroll
    for (int s2 = 0; s2 < CS; ++s2) {
      const int st = c * CS + s2;
      if (st < steps) {
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) {
          const i32x4 bv =
              *reinterpret_cast<const i32x4 *>(qs + (16 * sb + qn) * ld + 64 * st + 16 * grp);
#pragma unroll
          for (int i = 0; i < NT; ++i)
            acc[i][sb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ch.a[i][s2], bv, acc[i][sb], 0, 0, 0);
        }
      }
    }
    if (c != n_chunks - 1) return;
    const int tb = 64 * (wave + kWaves * j);                   // block start within the range
    uint32_t m[NT][NSB];   // best of the lane's 4 tools of each tile
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const f32x4 sc = *reinterpret_cast<const f32x4 *>(tsc + tb + 16 * i + 4 * grp);
      // all ones for a tool of the registry, 0 past its end: an AND, where a selection became a branch
      // around every score (4096 tools x 32 queries of 384: 9.6 against 7.7 us)
      uint32_t in[4];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        in[r] = (uint32_t)((t_begin + tb + 16 * i + 4 * grp + r - t_end) >> 31);
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) {
        uint32_t x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
          x[r] = score_order(((float)acc[i][sb][r] * sc[r]) * sq[sb]) & in[r];
        m[i][sb] = umax(umax(x[0], x[1]), umax(x[2], x[3]));
      }
    }
    // over the column's 4 lanes; lane group grp ends with tile 2 (grp & 1) + (grp >> 1)
    const int tile = ((t_begin + tb) >> 4) + 2 * (grp & 1) + (grp >> 1);
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) {
      const auto p01 = __builtin_amdgcn_permlane32_swap(m[0][sb], m[1][sb], false, false);
      const auto p23 = __builtin_amdgcn_permlane32_swap(m[2][sb], m[3][sb], false, false);
      const auto p = __builtin_amdgcn_permlane16_swap(umax(p01[0], p01[1]), umax(p23[0], p23[1]),
                                                      false, false);
      const int q = q0 + 16 * sb + qn;
      if (q < a.n_queries) a.tile_max[(size_t)q * a.tile_ld + tile] = umax(p[0], p[1]);
    }
  };
  if (total > 0) {
    int u = 0;
    for (;;) {
      load_chunk(u + 1, b1);
      step(u, b0);
      if (++u >= total) break;
      load_chunk(u + 1, b0);
      step(u, b1);
      if (++u >= total) break;
    }
  }
}

// ---- batches: pass 2, one workgroup per query.  The KT best tiles: every four threads take the best
// of their share, the KT-th best of those bounds the KT-th best tile from below, and the tiles at or
// above it (all in the at most KT quads whose own best reaches it, at most KT of each thread
// counting) are ranked by counting.  Then one MFMA chain per selected tile scores its tools with the query in
// every column, and the KT x 16 candidates are ranked by counting.  Latency-bound: a few dependent
// round trips, with all loads of each in flight together.
template <int KT>
__global__ __launch_bounds__(256) void slb_select_kernel(SlbArgs a) {
  constexpr int kGroups = 64;              // thread quads
  __shared__ __align__(16) uint64_t keys[16 * KT > kGroups ? 16 * KT : kGroups];
  __shared__ __align__(16) uint64_t hits[4 * KT * KT];
  __shared__ uint64_t floor_key;
  __shared__ uint64_t sorted[KT];
  __shared__ int sel[KT];
  __shared__ int n_hits;
  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  const int n_tiles = (a.n_tools + 15) / 16;
  const uint32_t *tm = a.tile_max + (size_t)q * a.tile_ld;     // tile_ld: a multiple of 4
  // a thread's share: quads of tiles tid, tid + 256, ..; the first kHeld stay in registers
  constexpr int kHeld = 4;
  u32x4 held[kHeld];
#pragma unroll
  for (int i = 0; i < kHeld; ++i) {
    const int t = 4 * tid + 1024 * i;
    held[i] = *reinterpret_cast<const u32x4 *>(tm + (t < a.tile_ld ? t : 0));
  }
  if (tid == 0) {
    floor_key = 0;
    n_hits = 0;
  }
  if (tid < KT) {
    sorted[tid] = 0;
    sel[tid] = -1;
  }
  // key of a tile: its best score, then the lower tile
  auto tile_key = [&](uint32_t ord, int t) -> uint64_t {
    return t < n_tiles ? ((uint64_t)ord << 32) | (0xFFFFFFFFu - (uint32_t)t) : 0;
  };
  auto each_tile = [&](auto f) {
#pragma unroll
    for (int i = 0; i < kHeld; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) f(tile_key(held[i][e], 4 * tid + 1024 * i + e));
#pragma unroll 4
    for (int t = 4 * tid + 1024 * kHeld; t < a.tile_ld; t += 1024) {
      const u32x4 v = *reinterpret_cast<const u32x4 *>(tm + t);
#pragma unroll
      for (int e = 0; e < 4; ++e) f(tile_key(v[e], t + e));
    }
  };
  uint64_t mine = 0;
  each_tile([&](uint64_t key) { mine = key > mine ? key : mine; });
  uint64_t best4 = mine;                   // of the quad's threads
#pragma unroll
  for (int off = 1; off < 4; off <<= 1) {
    const uint64_t o = shfl_xor_u64(best4, off);
    best4 = o > best4 ? o : best4;
  }
  if ((tid & 3) == 0) keys[tid >> 2] = best4;
  __syncthreads();
  auto rank_in = [&](const uint64_t *list, int n, uint64_t key) {
    int r = 0;
#pragma unroll 8
    for (int i = 0; i < n; i += 2) {       // an even number of keys, 16-byte aligned
      const u32x4 p = *reinterpret_cast<const u32x4 *>(list + i);
      r += (((uint64_t)p[1] << 32) | p[0]) > key ? 1 : 0;
      r += (((uint64_t)p[3] << 32) | p[2]) > key ? 1 : 0;
    }
    return r;
  };
  if (tid < kGroups) {
    const uint64_t key = keys[tid];
    if (key != 0 && rank_in(keys, kGroups, key) == KT - 1) floor_key = key;
  }
  __syncthreads();
  const uint64_t fl = floor_key;           // 0: fewer than KT quads have a tile
  if (mine != 0 && mine >= fl) {
    uint64_t b[KT];
#pragma unroll
    for (int j = 0; j < KT; ++j) b[j] = 0;
    each_tile([&](uint64_t key) { insert<KT>(b, key >= fl ? key : 0); });
    int n = 0;
#pragma unroll
    for (int j = 0; j < KT; ++j) n += b[j] != 0;
    const int at = atomicAdd(&n_hits, n);  // at most KT quads, 4 threads, KT tiles each
#pragma unroll
    for (int j = 0; j < KT; ++j)
      if (b[j] != 0) hits[at + j] = b[j];
  }
  __syncthreads();
  const int nh = n_hits;
  if (tid < nh) {                          // nh <= 4 KT KT <= 256
    const uint64_t key = hits[tid];
    int r = 0;
    for (int i = 0; i < nh; ++i) r += hits[i] > key;
    if (r < KT) sel[r] = (int)(0xFFFFFFFFu - (uint32_t)key);
  }
  __syncthreads();

  // ---- tools of the selected tiles: wave w takes places w, w + 4, ..
  const int dim = a.dim, steps = dim / 64;
  const float sq = a.query_scale[q];
  const int8_t *qrow = a.queries + (size_t)q * dim + 16 * grp;
  constexpr int TW = (KT + kWaves - 1) / kWaves;
  constexpr int CS = 8;                    // 64-byte steps loaded together
  int tile[TW];
  const int8_t *trow[TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int place = wave + kWaves * i;
    tile[i] = place < KT ? sel[place] : -1;
    trow[i] = a.tools + (size_t)min(16 * max(tile[i], 0) + qn, a.n_tools - 1) * dim + 16 * grp;
  }
  if (tile[0] >= 0) {                      // wave-uniform
    float st[TW];
#pragma unroll
    for (int i = 0; i < TW; ++i)
      st[i] = a.tool_scale[min(16 * max(tile[i], 0) + 4 * grp + (qn & 3), a.n_tools - 1)];
    i32x4 acc[TW];
#pragma unroll
    for (int i = 0; i < TW; ++i) acc[i] = i32x4{0, 0, 0, 0};
    for (int s0 = 0; s0 < steps; s0 += CS) {
      i32x4 bv[CS], av[TW][CS];
#pragma unroll
      for (int e = 0; e < CS; ++e) {       // steps past the end re-read the last one, unused
        const int off = 64 * min(s0 + e, steps - 1);
        bv[e] = *reinterpret_cast<const i32x4 *>(qrow + off);
#pragma unroll
        for (int i = 0; i < TW; ++i) av[i][e] = *reinterpret_cast<const i32x4 *>(trow[i] + off);
      }
#pragma unroll
      for (int e = 0; e < CS; ++e)
        if (s0 + e < steps) {
#pragma unroll
          for (int i = 0; i < TW; ++i)
            acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[i][e], bv[e], acc[i], 0, 0, 0);
        }
    }
    // all columns hold the query: lane qn < 4 of a group gives tool 4 grp + qn
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const int place = wave + kWaves * i;
      const int t = 16 * tile[i] + 4 * grp + qn;
      const int dot = qn == 0 ? acc[i][0] : qn == 1 ? acc[i][1] : qn == 2 ? acc[i][2] : acc[i][3];
      if (qn < 4 && place < KT) {
        uint64_t key = 0;
        if (tile[i] >= 0 && t < a.n_tools)
          key = cand_key(((float)dot * st[i]) * sq, t);
        keys[16 * place + 4 * grp + qn] = key;
      }
    }
  } else if (lane < 16) {
#pragma unroll
    for (int i = 0; i < TW; ++i)
      if (wave + kWaves * i < KT) keys[16 * (wave + kWaves * i) + lane] = 0;
  }
  __syncthreads();
  if (tid < 16 * KT) {
    const uint64_t key = keys[tid];
    if (key != 0) {
      const int r = rank_in(keys, 16 * KT, key);
      if (r < KT) sorted[r] = key;
    }
  }
  __syncthreads();
  if (tid < a.k) {
    a.top_idx[(size_t)q * a.k + tid] = cand_idx(sorted[tid]);
    a.top_score[(size_t)q * a.k + tid] = cand_score(sorted[tid]);
  }
  if (tid == 0) {
    // fewer than two tools: nothing to confuse the best one with
    const float m = sorted[1] == 0 ? INFINITY : cand_score(sorted[0]) - cand_score(sorted[1]);
    a.margin[q] = m;
    a.route[q] = m > a.tau ? 1 : 0;
  }
}

// One wave per query: the best KT of the ranges' lists, then the gate.
template <int KT>
__global__ __launch_bounds__(64) void slb_merge_kernel(SlbArgs a) {
  const int q = blockIdx.x, lane = threadIdx.x;
  uint64_t f[KT];
  wave_select<KT>(a.part + (size_t)q * a.n_ranges * KT, a.n_ranges * KT, lane, f);
  write_final<KT>(a, q, f, lane);
}

// Symmetric per-row INT8 quantisation: one wave per row; scale = max |x| / 127, code =
// x / scale rounded to nearest-even (IEEE fp32 division), |code| <= 127; a zero row gets scale 0.
__device__ __forceinline__ int quant_code(float x, float s) {
  const float c = s > 0.f ? rintf(x / s) : 0.f;
  return (int)fminf(fmaxf(c, -127.f), 127.f);
}
// QUADS: rows of 65 to 1024 features in whole, aligned float4s: the row is read once, all its loads
// in flight together, and stays in registers; else two passes, a feature per lane at a time, which is
// the faster way where a lane has one feature anyway (100000 rows of 64: 18.6 us, as quads 23.7; of 128
// 27.0 and 24.4).  The loads' latency bounds a small batch: 256 rows of 768: 8.4 -> 4.2 us; a
// registry of 65536 rows: 126 -> 52 us.
template <bool QUADS>
__global__ __launch_bounds__(256) void slb_quantize_kernel(const float *x, int32_t n, int32_t dim,
                                                           int8_t *q, float *scale) {
  constexpr int NV = 4;                    // float4s a lane holds
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const float *xr = x + (size_t)row * dim;
  int8_t *qr = q + (size_t)row * dim;
  float m = 0.f;
  f32x4 v[NV];
  if constexpr (QUADS) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int j = 4 * (lane + 64 * i);
      v[i] = j < dim ? *reinterpret_cast<const f32x4 *>(xr + j) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) m = fmaxf(m, fabsf(v[i][e]));
  } else {
    for (int j = lane; j < dim; j += 64) m = fmaxf(m, fabsf(xr[j]));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  const float s = m / 127.0f;
  if (lane == 0) scale[row] = s;
  if constexpr (QUADS) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int j = 4 * (lane + 64 * i);
      if (j >= dim) break;
      uint32_t w = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) w |= (uint32_t)(quant_code(v[i][e], s) & 0xff) << (8 * e);
      *reinterpret_cast<uint32_t *>(qr + j) = w;
    }
  } else {
    for (int j = lane; j < dim; j += 64) qr[j] = (int8_t)quant_code(xr[j], s);
  }
}

}  // namespace

namespace {
// Which kernels serve a scan.
enum class Path {
  kScan,    // slb_scan_kernel: 16-query blocks, ranges of tools over the workgroups for one block
  kTiles,   // slb_max_kernel, slb_select_kernel
  kLists,   // slb_block_kernel: 64-query blocks with a sorted list per lane
};
constexpr int kScanQueries = 16;          // one 16-query block
constexpr int32_t kOneRangeTools = 256;   // tools of one range of the scan kernel: no second launch
constexpr int kBlockQueries = 16 * kSubBlocks;
constexpr int64_t kBlockWgs = 512;        // batches: two resident workgroups per CU
constexpr int64_t kBlockMaxRange = 32;    // 64-tool blocks per range (its scales sit in LDS)
// Tile maxima of one pass over the registry: the batch goes in chunks of whole query blocks that
// stay within this (a registry of a million tools takes 256 queries a pass).
constexpr int64_t kTileMaxBytes = (int64_t)64 << 20;

// The tile kernels score a query's best tiles again, at 16 KT rows of `dim` bytes: their time grows with
// the queries where the lists' grows with queries x tools, so from a few thousand queries on the lists
// win over small registries, the sooner the fewer candidates are kept and the longer the rows are
// (dim 768, lists against tiles, us: 2048 queries over 300 tools k 2 23 : 31, k 3 32 : 37, k 8 67 : 53; 4096
// over 5000 53 : 74, 72 : 87, 138 : 119; 16384 over 8192 218 : 292, 274 : 347, 441 : 475; 65536 over 300
// 71 : 425, 97 : 654, 191 : 1150; 256 over 3000 22 : 19, 31 : 19, 65 : 23).
bool lists_win(int32_t n_tools, int32_t n_queries, int32_t dim, int32_t k) {
  const bool short_rows = dim < 512;
  const int64_t q = n_queries, t = n_tools;
  if (k <= 2)
    return short_rows ? q >= 2560 && t <= 4096 : q >= 1280 && t <= 16 * q && t <= 32768;
  if (k <= 4)
    return short_rows ? q >= 4096 && 2 * t <= q && t <= 4096 : q >= 1400 && t <= 4 * q && t <= 16384;
  return short_rows ? q >= 8192 && 4 * t <= q && t <= 4096 : q >= 3000 && t <= q - 2000 && t <= 8192;
}

// A registry of one range: the scan kernel reads its tools for every 16 queries, the list kernel for
// every 64, which pays with many queries and long rows (250 tools, lists against scan, us: dim 768, 65536
// queries k 2 53 : 97, k 3 73 : 101, k 8 159 : 125, 16384 k 3 30 : 31, 4096 k 3 29 : 14; dim 1024, 4096 k 3
// 36 : 41; dim 256, 65536 k 3 56 : 43).
bool lists_win_one_range(int32_t n_tools, int32_t n_queries, int32_t dim, int32_t k) {
  const int32_t t = n_tools, q = n_queries;
  if (k > 4) return dim > 768 && t > 192 && q >= 32768;
  if (dim > 768) return t > 64 && q >= (t > 128 ? 4096 : 16384);
  if (dim >= 512) return (t > 128 && q >= 16384) || (k <= 2 && t > 64 && q >= 32768);
  return dim > 256 && t > 128 && q >= 32768;
}

Path path_of(int32_t n_tools, int32_t n_queries, int32_t dim, int32_t k) {
  if (n_queries <= kScanQueries) return Path::kScan;
  if (n_tools <= kOneRangeTools)
    return lists_win_one_range(n_tools, n_queries, dim, k) ? Path::kLists : Path::kScan;
  return lists_win(n_tools, n_queries, dim, k) ? Path::kLists : Path::kTiles;
}
int64_t tile_ld_of(int32_t n_tools) { return ((int64_t)n_tools + 63) / 64 * 4; }
int32_t chunk_queries(int32_t n_tools, int32_t n_queries) {
  const int64_t fit = kTileMaxBytes / (tile_ld_of(n_tools) * 4) / kBlockQueries * kBlockQueries;
  const int64_t c = fit < kBlockQueries ? kBlockQueries : fit;
  return (int32_t)(c < n_queries ? c : n_queries);
}
// Tools per range of a batched pass: about kBlockWgs workgroups, 4 to kBlockMaxRange 64-tool
// blocks per range (at least one block per wave).
int32_t block_range_tools(int32_t n_tools, int32_t n_queries) {
  const int64_t q_blocks = ((int64_t)n_queries + kBlockQueries - 1) / kBlockQueries;
  const int64_t blocks = ((int64_t)n_tools + 63) / 64;
  int64_t per = (blocks * q_blocks + kBlockWgs - 1) / kBlockWgs;
  if (per < 4) per = 4;
  if (per > kBlockMaxRange) per = kBlockMaxRange;
  return (int32_t)(per * 64);
}

// Ranges of the scan and list kernels and the tools of each.
void ranges_of(Path path, int32_t n_tools, int32_t n_queries, int32_t &n_ranges, int32_t &range_tools) {
  if (path == Path::kLists) {
    range_tools = block_range_tools(n_tools, n_queries);
  } else {
    const int64_t tiles = ((int64_t)n_tools + 63) / 64;                 // 64-tool units
    // at least 256 tools per range, at most 256 ranges (the merge reads 8 candidates of each)
    const int64_t nr = std::min<int64_t>((tiles + 3) / 4, 256);
    range_tools = (int32_t)((tiles + nr - 1) / nr * 64);
  }
  n_ranges = (int32_t)(((int64_t)n_tools + range_tools - 1) / range_tools);
}
}  // namespace

size_t slb_workspace_bytes(int32_t n_tools, int32_t n_queries, int32_t dim, int32_t k) {
  const Path path = path_of(n_tools, n_queries, dim, k);
  if (path == Path::kTiles)
    return (size_t)chunk_queries(n_tools, n_queries) * tile_ld_of(n_tools) * sizeof(uint32_t);
  int32_t nr, rt;
  ranges_of(path, n_tools, n_queries, nr, rt);
  if (nr <= 1) return 0;
  return (size_t)n_queries * nr * kTop * sizeof(uint64_t);
}

hipError_t launch_slb_quantize(const float *x, int32_t n, int32_t dim, int8_t *q, float *scale,
                               hipStream_t stream) {
  const bool quads = dim % 4 == 0 && dim > 64 && dim <= 1024 && (uintptr_t)x % 16 == 0 && (uintptr_t)q % 4 == 0;
  if (quads)
    hipLaunchKernelGGL(slb_quantize_kernel<true>, dim3((n + 3) / 4), dim3(256), 0, stream, x, n, dim,
                       q, scale);
  else
    hipLaunchKernelGGL(slb_quantize_kernel<false>, dim3((n + 3) / 4), dim3(256), 0, stream, x, n, dim,
                       q, scale);
  return hipGetLastError();
}

hipError_t launch_slb_scan(const SlbLaunch &p, hipStream_t stream) {
  SlbArgs a{};
  a.tools = p.tools;
  a.tool_scale = p.tool_scale;
  a.queries = p.queries;
  a.query_scale = p.query_scale;
  a.n_tools = p.n_tools;
  a.n_queries = p.n_queries;
  a.dim = p.dim;
  a.k = p.k;
  a.tau = p.tau;
  a.top_idx = p.top_idx;
  a.top_score = p.top_score;
  a.margin = p.margin;
  a.route = p.route;
  const int kt = p.k <= 2 ? 2 : p.k <= 4 ? 4 : 8;
  const Path path = path_of(p.n_tools, p.n_queries, p.dim, p.k);
  if (path == Path::kTiles) {
    a.tile_max = reinterpret_cast<uint32_t *>(p.workspace);
    a.tile_ld = (int32_t)tile_ld_of(p.n_tools);
    const int32_t chunk = chunk_queries(p.n_tools, p.n_queries);
    for (int32_t q0 = 0; q0 < p.n_queries; q0 += chunk) {
      a.n_queries = p.n_queries - q0 < chunk ? p.n_queries - q0 : chunk;
      a.queries = p.queries + (size_t)q0 * p.dim;
      a.query_scale = p.query_scale + q0;
      a.top_idx = p.top_idx + (size_t)q0 * p.k;
      a.top_score = p.top_score + (size_t)q0 * p.k;
      a.margin = p.margin + q0;
      a.route = p.route + q0;
      a.n_qblocks = (a.n_queries + kBlockQueries - 1) / kBlockQueries;
      a.range_tools = block_range_tools(p.n_tools, a.n_queries);
      a.n_ranges = (int32_t)(((int64_t)p.n_tools + a.range_tools - 1) / a.range_tools);
      const size_t lds = (size_t)kBlockQueries * (p.dim + kQPad) +
                         (size_t)a.range_tools * sizeof(float);
      if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(slb_max_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)lds);
        if (e != hipSuccess) return e;
      }
      const uint32_t wgs = ((uint32_t)a.n_ranges * (uint32_t)a.n_qblocks + 7) / 8 * 8;
      hipLaunchKernelGGL(slb_max_kernel, dim3(wgs), dim3(256), lds, stream, a);
      const dim3 sgrid(a.n_queries);
      if (kt == 2) hipLaunchKernelGGL(slb_select_kernel<2>, sgrid, dim3(256), 0, stream, a);
      else if (kt == 4) hipLaunchKernelGGL(slb_select_kernel<4>, sgrid, dim3(256), 0, stream, a);
      else hipLaunchKernelGGL(slb_select_kernel<8>, sgrid, dim3(256), 0, stream, a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  ranges_of(path, p.n_tools, p.n_queries, a.n_ranges, a.range_tools);
  if (a.n_ranges > 1) a.part = reinterpret_cast<uint64_t *>(p.workspace);
  if (path == Path::kLists) {
    const size_t stage = (size_t)kBlockQueries * (p.dim + kQPad) + (size_t)a.range_tools * sizeof(float);
    const size_t merge = (size_t)kWaves * kBlockQueries * kTop * 8;
    const size_t lds = stage > merge ? stage : merge;
    const dim3 grid(a.n_ranges, (p.n_queries + kBlockQueries - 1) / kBlockQueries);
    auto run = [&](auto kernel, auto merge_kernel) -> hipError_t {
      if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
      }
      hipLaunchKernelGGL(kernel, grid, dim3(256), lds, stream, a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess || a.n_ranges <= 1) return e;
      hipLaunchKernelGGL(merge_kernel, dim3(p.n_queries), dim3(64), 0, stream, a);
      return hipGetLastError();
    };
    return kt == 2   ? run(slb_block_kernel<2>, slb_merge_kernel<2>)
           : kt == 4 ? run(slb_block_kernel<4>, slb_merge_kernel<4>)
                     : run(slb_block_kernel<8>, slb_merge_kernel<8>);
  }
  // one 16-query block, or several over a registry of one range
  const dim3 grid((p.n_queries + 15) / 16, a.n_ranges);
  const size_t stage = (size_t)16 * (p.dim + kQPad);
  const size_t merge = (size_t)kWaves * 16 * kTop * 8;
  const size_t lds = stage > merge ? stage : merge;
  const int steps = p.dim / 64;
#define NEXUS_SLB(S_, K_) \
  hipLaunchKernelGGL((slb_scan_kernel<S_, K_>), grid, dim3(256), lds, stream, a)
#define NEXUS_SLB_S(K_)                      \
  do {                                       \
    if (steps <= 4) NEXUS_SLB(4, K_);        \
    else if (steps <= 8) NEXUS_SLB(8, K_);   \
    else if (steps <= 12) NEXUS_SLB(12, K_); \
    else NEXUS_SLB(16, K_);                  \
  } while (0)
  if (kt == 2) NEXUS_SLB_S(2);
  else if (kt == 4) NEXUS_SLB_S(4);
  else NEXUS_SLB_S(8);
#undef NEXUS_SLB_S
#undef NEXUS_SLB
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_ranges <= 1) return e;
  if (kt == 2) hipLaunchKernelGGL(slb_merge_kernel<2>, dim3(p.n_queries), dim3(64), 0, stream, a);
  else if (kt == 4) hipLaunchKernelGGL(slb_merge_kernel<4>, dim3(p.n_queries), dim3(64), 0, stream, a);
  else hipLaunchKernelGGL(slb_merge_kernel<8>, dim3(p.n_queries), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace nexus
