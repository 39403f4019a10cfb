// fp32 causal grouped-query suffix attention (Sec. III-A) for f32 caches: fp32 MFMA throughout
// (products, accumulation, softmax), no workspace.
//
// A workgroup serves one KV head and 16 rows of its group, a row being one (query, query head of
// the group) pair in query-major order, so the G heads of a group share the keys and values they
// read.  Its NW waves take the 16-key pages round-robin and merge their (m, l, O) through LDS at
// the end, in wave order: the key axis is split inside the workgroup, which fills the chip at a
// few hundred rows without partials in memory (f32 launches have no workspace).
//
// Per wave and page, v_mfma_f32_16x16x4_f32 (lane = column col = lane % 16, group grp = lane / 16):
//   S^T (16 keys x 16 rows) = K.Q^T.  The order of the k index is free, so lane (col, grp) loads
//     features 16 c + 4 grp .. +3 of key row col as one 16-byte load, and register j of it is the
//     operand of step (c, j); Q sits in registers in the same layout.  Four accumulators (one per
//     j) keep the chains independent.
//   O^T (features x 16 rows) += V^T.P^T.  Lane (col, grp) holds the scores of keys 4 grp + i, which
//     is the B operand of step i = keys {4 grp + i} as it stands.  V row-major: the lane loads
//     features 64 u + 4 col .. +3 of key 4 grp + i, so register r feeds the output tile whose row m
//     is feature 64 u + 4 m + r; V transposed: keys 4 grp .. +3 of feature 16 ft + col, register i
//     feeding step i.  No operand crosses lanes and nothing is staged in LDS.
// A page's V is in flight under its score products and the next page's K under its output
// products, each in one set of registers.  Bound: the fp32 matrix rate (one wave reads 8 D x 16
// bytes per 16 D/2 matrix instructions of 32 cycles, about half of what L2 delivers) for launches
// that fill the chip, latency below.  96 queries x 40 heads over 1120 keys of head_dim 128 (2.1
// GFLOP, 13 us at the fp32 matrix rate): 32 us against 754 us for a workgroup per (query, head)
// with scalar products; error against 64 bits 4.5e-7 against 1.1e-6.
#include "attn_common.h"
#include "launch.h"

#include <stdint.h>

#include <algorithm>
#include <type_traits>

namespace nexus {

struct F32SeqTable {
  AttnSeq seq[kMaxSeqs];
  int32_t tile_begin[kMaxSeqs + 1];   // prefix sums of the sequences' 16-row tiles per KV head
};

struct F32Args {
  const float *q;
  float *out;
  const float *kc, *vc;               // layer bases
  const int32_t *map;
  int32_t n_kv_heads, n_q_heads, group, n_seqs;
  int32_t first_tile;                 // of this launch
  int64_t n_cols;                     // transposed V row length
  float scale, softcap;
};

template <int D, int NW, bool VT, bool CAP>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(const F32Args a, const F32SeqTable tab) {
  constexpr int NC = D >= 16 ? D / 16 : 1;        // 16-feature chunks of a key row
  constexpr int NU = D >= 64 ? D / 64 : 1;        // 64-feature chunks of a row-major value row
  constexpr int NT = VT ? NC : 4 * NU;            // 16-feature output tiles
  constexpr int NV = VT ? NC : 4 * NU;            // 16-byte V loads of a lane per page
  constexpr int LD = D + 4;                       // padded merge row (floats)
  __shared__ __align__(16) float mo[NW][16][LD];
  __shared__ float mml[NW][16][2];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;
  const int kvh = blockIdx.x % a.n_kv_heads;
  const int t = a.first_tile + blockIdx.x / a.n_kv_heads;
  int b = 0;
  while (b + 1 < a.n_seqs && t >= tab.tile_begin[b + 1]) ++b;
  const AttnSeq sq = tab.seq[b];
  const int G = a.group;
  // later rows see more keys: longest tiles first
  const int tl = tab.tile_begin[b + 1] - 1 - t;
  const int n_rows = sq.len * G;
  const int row0 = tl * 16;
  const int row = min(row0 + col, n_rows - 1);
  const int qi = row / G;
  const int pos = (int)sq.n_past + qi;                                   // this lane's row
  const int pos_lo = (int)sq.n_past + row0 / G;                          // earliest of the tile
  const int n_keys = (int)sq.n_past + min(row0 + 15, n_rows - 1) / G + 1;
  const int n_pages = (n_keys + kPage - 1) / kPage;
  const int64_t qoff = ((int64_t)(sq.q_start + qi) * a.n_q_heads + kvh * G + (row - qi * G)) * D;

  f32x4 q[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    q[c] = 16 * c + 4 * grp < D
               ? *reinterpret_cast<const f32x4 *>(a.q + qoff + 16 * c + 4 * grp)
               : f32x4{0.f, 0.f, 0.f, 0.f};

  // Transposed V addresses: a uniform row-tile base plus a lane offset, which 32 bits hold (in
  // bytes) from head_dim 32 on, because a layer has less than 2^31 elements.
  using VOff = typename std::conditional<(D >= 32), uint32_t, uint64_t>::type;
  auto at = [](const float *base, VOff elems) {
    return reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + elems * (VOff)4);
  };
  // Loads of logical page p at physical page phys.  Rows past the tile's last key re-read that
  // key (masked later); transposed V slots past it are zeroed before use.
  f32x4 kr[NC], vr[NV];
  auto load_k = [&](int p, int32_t phys) {
    const float *kp = a.kc + ((int64_t)phys * a.n_kv_heads + kvh) * (kPage * D);
    const int off = min(col, n_keys - 1 - kPage * p) * D + 4 * grp;
#pragma unroll
    for (int c = 0; c < NC; ++c)
      kr[c] = 16 * c + 4 * grp < D ? *reinterpret_cast<const f32x4 *>(kp + off + 16 * c)
                                   : f32x4{0.f, 0.f, 0.f, 0.f};
  };
  auto load_v = [&](int p, int32_t phys) {
    if constexpr (!VT) {
      const float *vp = a.vc + ((int64_t)phys * a.n_kv_heads + kvh) * (kPage * D);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int off = min(4 * grp + i, n_keys - 1 - kPage * p) * D + 4 * col;
#pragma unroll
        for (int u = 0; u < NU; ++u)
          vr[i * NU + u] = 64 * u + 4 * col < D
                               ? *reinterpret_cast<const f32x4 *>(vp + off + 64 * u)
                               : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    } else {
      const float *vp = a.vc + (int64_t)kvh * D * a.n_cols + (int64_t)phys * kPage;
      const VOff off = (VOff)col * (VOff)a.n_cols + 4 * grp;
#pragma unroll
      for (int ft = 0; ft < NC; ++ft)
        vr[ft] = 16 * ft + col < D
                     ? *reinterpret_cast<const f32x4 *>(at(vp + (int64_t)(16 * ft) * a.n_cols, off))
                     : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  // feature of row 4 grp + e of output tile nt, for this lane
  auto feature = [&](int nt, int e) {
    return VT ? 16 * nt + 4 * grp + e : 64 * (nt >> 2) + 16 * grp + 4 * e + (nt & 3);
  };

  f32x4 o[NT];
#pragma unroll
  for (int n = 0; n < NT; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;   // running maximum of row col; this lane's share of its row sum

  // this wave's pages wave, wave + NW, ...: a page's V loads are in flight under its score
  // products, the next page's K loads under its output products (past the end the last page is
  // re-read, so that every step waits for the same loads)
  const int n_mine = n_pages > wave ? (n_pages - wave + NW - 1) / NW : 0;
  auto page_of = [&](int k) { return wave + NW * min(k, n_mine - 1); };
  int32_t phys = 0, phys_next = 0;
  if (n_mine > 0) {
    phys = a.map[page_of(0)];
    phys_next = a.map[page_of(1)];
    load_k(page_of(0), phys);
  }
  for (int it = 0; it < n_mine; ++it) {
    const int p = page_of(it);
    load_v(p, phys);
    const int32_t phys_after = a.map[page_of(it + 2)];
    f32x4 s4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s4[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        s4[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[c][j], q[c][j], s4[j], 0, 0, 0);
    load_k(page_of(it + 1), phys_next);
    const int key0 = kPage * p + 4 * grp;
    const bool diag = kPage * p + kPage - 1 > pos_lo;   // some row does not see the whole page
    float x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = ((s4[0][i] + s4[1][i]) + (s4[2][i] + s4[3][i])) * a.scale;
      if constexpr (CAP) x[i] = a.softcap * tanhf(x[i] / a.softcap);
      if (diag && key0 + i > pos) x[i] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (__builtin_amdgcn_ballot_w64(mx > m)) {
      const float m_new = fmaxf(m, mx);
      // a row that has met no visible key yet has nothing to rescale
      const float alpha = m == -INFINITY ? 0.f : __expf(m - m_new);
      l *= alpha;
#pragma unroll
      for (int n = 0; n < NT; ++n) o[n] *= alpha;
      m = m_new;
    }
    float pr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // exactly 0 for a masked key, also while its row has met no visible key (m = -inf); a NaN
      // score stays one
      pr[i] = x[i] == -INFINITY ? 0.f : __expf(x[i] - m);
      l += pr[i];
    }
    bool odd = false;
    if (diag) {
      if constexpr (VT) {
        const int keep = n_keys - key0;   // slots past the last key may hold anything
#pragma unroll
        for (int ft = 0; ft < NC; ++ft)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (i >= keep) vr[ft][i] = 0.f;
      }
#pragma unroll
      for (int n = 0; n < NV; ++n)
#pragma unroll
        for (int e = 0; e < 4; ++e) odd |= !(fabsf(vr[n][e]) <= 3.402823466e38f);
    }
    if (__builtin_amdgcn_ballot_w64(odd)) {
      // A key that some rows of the tile do not see must not reach them even where its value
      // row holds an infinity or a NaN (0 x inf): such a page is taken row by row, with the values
      // that the row does not see set to 0.
#pragma unroll 1
      for (int r = 0; r < 16; ++r) {
        const int pos_r = (int)sq.n_past + min(row0 + r, n_rows - 1) / G;
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          f32x4 acc = o[n];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float va = VT ? vr[n][i] : vr[i * NU + (n >> 2)][n & 3];
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(key0 + i > pos_r ? 0.f : va, pr[i], acc, 0,
                                                       0, 0);
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) o[n][e] = col == r ? acc[e] : o[n][e];
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < NT; ++n) {
          const float va = VT ? vr[n][i] : vr[i * NU + (n >> 2)][n & 3];
          o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(va, pr[i], o[n], 0, 0, 0);
        }
    }
    phys = phys_next;
    phys_next = phys_after;
  }

  // merge the waves' states: each stores its own, then thread x forms 4 features of one row
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (grp == 0) {
    mml[wave][col][0] = m;
    mml[wave][col][1] = l;
  }
#pragma unroll
  for (int n = 0; n < (VT ? NT : NU); ++n)
#pragma unroll
    for (int e = 0; e < (VT ? 1 : 4); ++e) {
      const int d = VT ? feature(n, 0) : feature(4 * n, e);
      if (d < D)
        *reinterpret_cast<f32x4 *>(&mo[wave][col][d]) =
            VT ? o[n] : f32x4{o[4 * n][e], o[4 * n + 1][e], o[4 * n + 2][e], o[4 * n + 3][e]};
    }
  __syncthreads();
  for (int x = threadIdx.x; x < 16 * (D / 4); x += 64 * NW) {
    const int r = x / (D / 4), d = 4 * (x % (D / 4));
    if (row0 + r >= n_rows) continue;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, mml[w][r][0]);
    float ls = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float mw = mml[w][r][0], lw = mml[w][r][1];
      // a wave that saw no visible key of the row has m = -inf and l = 0 (or NaN, which must show)
      if (mw == -INFINITY && lw == 0.f) continue;
      const float wt = mw == -INFINITY ? 1.f : __expf(mw - M);
      ls += wt * lw;
      acc += *reinterpret_cast<const f32x4 *>(&mo[w][r][d]) * wt;
    }
    const int rr = row0 + r, i = rr / G;
    *reinterpret_cast<f32x4 *>(a.out + ((int64_t)(sq.q_start + i) * a.n_q_heads + kvh * G +
                                        (rr - i * G)) * D + d) = acc / ls;
  }
}

namespace {

template <int D, int NW>
hipError_t launch_f32(F32Args a, const F32SeqTable &tab, int32_t tiles, bool vt, hipStream_t stream) {
  const bool cap = a.softcap > 0.f;
  // a grid dimension holds less than 2^32 threads: more tiles than that go in several launches
  const int32_t most = std::max(1, (int32_t)(UINT32_MAX / (64 * NW) / (uint32_t)a.n_kv_heads));
  for (; a.first_tile < tiles; a.first_tile += most) {
    const dim3 grid((uint32_t)std::min(tiles - a.first_tile, most) * a.n_kv_heads);
#define NEXUS_F32(VT_, CAP_) \
  hipLaunchKernelGGL((attn_f32_kernel<D, NW, VT_, CAP_>), grid, dim3(64 * NW), 0, stream, a, tab)
    if (vt) {
      if (cap) NEXUS_F32(true, true); else NEXUS_F32(true, false);
    } else {
      if (cap) NEXUS_F32(false, true); else NEXUS_F32(false, false);
    }
#undef NEXUS_F32
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (most > tiles - a.first_tile) break;   // (first_tile + most might not fit)
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_attention_f32(const AttnLaunch &p, hipStream_t stream) {
  const int64_t layer_elems = (int64_t)p.n_phys_pages * p.n_kv_heads * kPage * p.head_dim;
  F32Args a{};
  a.q = (const float *)p.q;
  a.out = (float *)p.out;
  a.kc = (const float *)p.cache_k + p.layer * layer_elems;
  a.vc = (const float *)p.cache_v + p.layer * layer_elems;
  a.map = p.map;
  a.n_kv_heads = p.n_kv_heads;
  a.n_q_heads = p.n_q_heads;
  a.group = p.n_q_heads / p.n_kv_heads;
  a.n_seqs = p.n_seqs;
  a.n_cols = (int64_t)p.n_phys_pages * kPage;
  a.scale = p.scale;
  a.softcap = p.softcap;
  F32SeqTable tab{};
  int32_t tiles = 0;
  for (int b = 0; b < p.n_seqs; ++b) {
    tab.seq[b] = p.seqs[b];
    tab.tile_begin[b] = tiles;
    tiles += (p.seqs[b].len * a.group + 15) / 16;
  }
  tab.tile_begin[p.n_seqs] = tiles;
  // 8 waves fit two to a SIMD up to head_dim 128 (Q, O, K and V of a page take 128 registers);
  // head_dim 256 needs twice that, so 4 waves, one to a SIMD
  switch (p.head_dim) {
    case 8: return launch_f32<8, 8>(a, tab, tiles, p.v_transposed, stream);
    case 16: return launch_f32<16, 8>(a, tab, tiles, p.v_transposed, stream);
    case 32: return launch_f32<32, 8>(a, tab, tiles, p.v_transposed, stream);
    case 64: return launch_f32<64, 8>(a, tab, tiles, p.v_transposed, stream);
    case 128: return launch_f32<128, 8>(a, tab, tiles, p.v_transposed, stream);
    case 256: return launch_f32<256, 4>(a, tab, tiles, p.v_transposed, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nexus
