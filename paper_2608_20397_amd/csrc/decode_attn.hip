// Decode-step attention over the paged cache: one new query token per sequence attends to every
// cached token of its own sequence (generation after the first token, over the spliced cache;
// scaled dot-product attention of Sec. III-A, soft-cap and transposed V of Sec. VI-B).
//
// Each sequence has its own page map and a device-resident length, so a decode loop can bump the
// lengths on the device and replay the same launch.  Keys are split into fixed runs of
// `split_pages` pages (flash-decoding); a workgroup handles one (sequence, KV head, query-head
// group of up to 16, split) and a second small kernel merges the splits.  The work is
// HBM-bound: each key and value row is read once per (sequence, KV head), shared by the G query
// heads of the group.
//
// bf16 (MFMA) kernel, per wave and 16-key page:
//   * S^T = K.Q^T on v_mfma_f32_16x16x32_bf16: lane l feeds key row l % 16, features
//     32 s + 8 (l / 16) .. +7 of step s straight from global memory (16 bytes); the query heads
//     of the group are the 16 columns (columns past G are zero).  Lane l then holds the scores
//     of keys 4 (l / 16) .. +3 for query column l % 16;
//   * online softmax in log2 units with a lazily moved reference (rescale only when a page's
//     maximum exceeds the reference by more than kDecSlack); P is rounded to bf16 and the row sums add
//     the rounded values;
//   * O^T += V^T.P^T on v_mfma_f32_16x16x32_bf16, two pages at a time: the scores are already in
//     the B-operand layout (keys 4 (l / 16) .. +3 of either page).  A transposed V cache gives the
//     A operand (4 consecutive keys of one feature) directly from global memory; a row-major V page
//     is staged in the wave's own LDS slot and read back with ds_read_b64_tr_b16 (in each 16-lane
//     group, output lane i receives element i % 4 of the 8 bytes that source lane 4e + i / 4 points
//     at).
// The 4 waves of a workgroup take pairs of the split's pages round-robin, loading the next pair
// into registers while computing the current one, and merge their (m, l, O) through LDS at the end.
// Key rows past the sequence end are never used: the last page's loads re-read the last valid
// row (row-major) or are zeroed (transposed V), and their scores are -inf.
#include "attn_common.h"
#include "attn_dma.h"
#include "launch_decode.h"

#include <stdint.h>

#include <algorithm>
#include <type_traits>

namespace nexus {

namespace {

constexpr int kDecWaves = 4;
// log2 units the reference may lag behind the running maximum.  A moved reference gives the key it
// moves to the probability 1, which bf16 holds exactly, and a few top keys carry much of the
// rounding error: 32 sequences of 17473 keys, relative error against 64 bits 2.20e-3 at a lag of
// 8, 2.08e-3 at 6, 2.04e-3 at 4 (2.15e-3 at 8 with pages taken one by one).
constexpr float kDecSlack = 6.0f;
constexpr int kMaxDecSplits = 1024; // splits per sequence at most (bounds the merge's loop)
constexpr int kMaxSplitPages = 2048;  // pages per split at most (page list in LDS)
constexpr int kMaxSharedPages = 1024; // pages per shared range at most (page list and masks in LDS)
constexpr int kMinRangePages = 16;    // and at least
constexpr int kMaxGroupSeqs = 32;     // sequences whose shared pages one workgroup serves
constexpr int64_t kSharedMinBytes = (int64_t)512 << 20;   // keys + values of all sequences
constexpr int kSharedStages = 4;      // ring of page pairs in LDS (shared pages)

struct DecodeArgs {
  const void *q;
  void *out;
  const void *kc;         // layer base of the K cache [NPP][Hkv][16][D]
  const void *vc;         // layer base of V: as K, or [Hkv][D][NPP * 16] when transposed
  const int32_t *maps;    // [n_seqs][map_stride]
  const int32_t *lens;    // [n_seqs]
  float *part;            // [n_seqs][Hq][max_splits][D] unnormalised split outputs
  float *part_ml;         // [n_seqs][Hq][max_splits][2] (reference m, row sum l)
  int32_t map_stride, max_len, n_q_heads, n_kv_heads, group, n_qgroups;
  int32_t split_pages, max_splits;      // max_splits: partial slots per row
  int32_t n_seqs;
  // shared pages (0 groups: none looked for): slots own_splits .. max_splits - 1 of a row belong
  // to the page ranges of its group
  int32_t n_groups, group_seqs, shared_splits, own_splits;
  int32_t share_pages;    // whole pages from which on a sequence is long enough to share them
  int32_t *flags;         // [n_seqs]: ranges of shared pages a sequence has partials of (the merge's use)
  uint32_t n_cols;        // transposed V: NPP * 16
  float scale_log2;       // scale * log2(e)
  float cap_in;           // scale / softcap
  float cap_out;          // softcap * log2(e)
};

__device__ __forceinline__ float max_x16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_x32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_x16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_x32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sequence length as the kernels read it: clamped to [0, max_len].
__device__ __forceinline__ int seq_len_of(const DecodeArgs &a, int b) {
  return min(max(a.lens[b], 0), a.max_len);
}

// 16-byte chunk c of row r of a staged V page lives at chunk c ^ vswz(r): the 16 rows of one
// transposed read (32 bytes each) and the 4 rows of one staging write cover distinct banks.
template <int D>
__device__ __forceinline__ int vswz(int r) {
  return D == 64 ? 2 * ((r >> 1) & 3) : 2 * (r & 7);
}

// Writes the partial (O unnormalised, m, l) of a lane's row; a negative row is skipped.
template <int D>
__device__ __forceinline__ void store_part(const DecodeArgs &a, int row, int slot_of_row,
                                           const f32x4 (&o)[D / 16], float m, float l, int grp) {
  if (row < 0) return;
  const size_t slot = (size_t)row * a.max_splits + slot_of_row;
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
    *reinterpret_cast<f32x4 *>(a.part + slot * D + 16 * t + 4 * grp) = o[t];
  if (grp == 0) {
    a.part_ml[2 * slot] = m;
    a.part_ml[2 * slot + 1] = l;
  }
}
// Marks a row's partial slot as empty.
__device__ __forceinline__ void store_empty(const DecodeArgs &a, int row, int slot_of_row, int grp) {
  if (row < 0 || grp != 0) return;
  const size_t slot = (size_t)row * a.max_splits + slot_of_row;
  a.part_ml[2 * slot] = -INFINITY;
  a.part_ml[2 * slot + 1] = 0.f;
}

// ---- pages shared between sequences (a warm prefix).  Consecutive sequences form groups of up to
// kMaxGroupSeqs.  Page p of two sequences of a group counts as shared when it is whole in both and both
// map it to one physical page; such pages are read once for all the group's sharers, every other page by
// its sequence alone.  To that end a page is compared with that of one sharer, the representative, whose
// own page counts when any other sharer's does.
// Whether a group shares is settled by looks at two pages, where it pays:
//   * half of its sequences or more have share_pages whole pages, their part of kSharedMinBytes / 2; below
//     that the caches serve the repeated reads, whatever the launch's bound (32 sequences of 500 tokens,
//     256 of them shared, in a launch for 17473: 18 us, through the shared pages 43; of 2100 tokens, 1050
//     shared: 49 and 40);
//   * they share the first half: 32 sequences of 17473 tokens that share 4096, 6144, 8192, 12800 tokens take
//     306, 275, 243, 202 us page by page and 322, 281, 243, 142 so.  The first look, at page
//     share_pages / 2, costs nothing: it is loaded with the lengths;
//   * every sequence that long shares, because one that does not takes as long as ever (31 of 32 sequences
//     on a prefix, one private: 176 us page by page, 196 so; the first one alone: 171, 185).
struct GroupState {
  int b0, n;          // first sequence, sequences
  int rep;            // representative (index in the group)
  int rep_full;       // its whole pages
  uint32_t sharers;   // sequences that share pages (the representative first); 0: nothing is shared
  int n_sh;           // their number
  bool by_split;      // order of the workgroups: splits vary slowest
};
// Lanes j and j + 32 hold the whole pages and page share_pages / 2 of sequence j of group g.
__device__ __forceinline__ GroupState group_state(const DecodeArgs &a, int g, int full, int32_t page) {
  GroupState s;
  s.b0 = g * a.group_seqs;
  s.n = min(a.group_seqs, a.n_seqs - s.b0);
  const int j = threadIdx.x & 31;
  auto which = [&](bool x) { return (uint32_t)__builtin_amdgcn_ballot_w64(x && j < s.n); };
  s.by_split = 2 * __popc(which(2 * (int64_t)full <= (int64_t)a.own_splits * a.split_pages)) > s.n;
  s.rep = s.rep_full = s.n_sh = 0;
  s.sharers = 0;
  const uint32_t large = which(full >= a.share_pages);
  if (__popc(large) < max(2, (s.n + 1) / 2)) return s;
  s.rep = __builtin_ctz(large);
  s.rep_full = __builtin_amdgcn_readlane(full, s.rep);
  if (large & ~which(page == __builtin_amdgcn_readlane(page, s.rep))) return s;
  const int half = s.rep_full / 2;
  const uint32_t longer = which(full > half);
  const int32_t x = a.maps[(size_t)(s.b0 + min(j, s.n - 1)) * a.map_stride + half];
  if (__popc(longer) < 2 || longer & ~which(x == __builtin_amdgcn_readlane(x, s.rep))) return s;
  s.sharers = longer;
  s.rep = __builtin_ctz(longer);
  s.rep_full = __builtin_amdgcn_readlane(full, s.rep);
  s.n_sh = __popc(longer);
  s.by_split = true;
  return s;
}

// Ranges that a group's shared pages are cut into and pages of each: one for each workgroup of the
// sharers (per KV head and query group), up to the partial slots, at least kMinRangePages pages.  Every
// sequence has a workgroup for each 2048 pages and a group two sharers, so no workgroup has two ranges.
__device__ __forceinline__ void shared_ranges(const DecodeArgs &a, const GroupState &gs, int &n_ranges,
                                              int &range_pages) {
  const int n = min(a.shared_splits, gs.n_sh * a.own_splits);
  range_pages = min(max((gs.rep_full + n - 1) / n, kMinRangePages), kMaxSharedPages);
  n_ranges = (gs.rep_full + range_pages - 1) / range_pages;
}

// 16-query column blocks of a wave that serves shared pages.
__host__ __device__ constexpr int shared_blocks(int head_dim) { return head_dim == 256 ? 2 : 3; }

// Place in a list of n entries that a thread's entry takes if it is appended, in thread order; n grows by
// the workgroup's entries.  Called by the whole workgroup; it holds barriers, the last of them after every
// thread has read the counts.
__device__ __forceinline__ int place(bool take, int &n, int32_t *wave_cnt) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t m = __builtin_amdgcn_ballot_w64(take);
  if (lane == 0) wave_cnt[wave] = __popcll(m);
  __syncthreads();
  int at = n;
#pragma unroll
  for (int w = 0; w < kDecWaves; ++w) {
    const int c = wave_cnt[w];
    if (w < wave) at += c;
    n += c;
  }
  __syncthreads();
  return at + __popcll(m & ((1ull << lane) - 1));
}

// The shared pages of one range (the representative's pages p_lo .. + n_range - 1), for the query heads hg
// of the group's sharers: one 16-query column block holds 16 / G of them (one when G > 16), the column
// blocks are dealt to the 4 waves and every wave reads every page.  Page pairs travel global -> LDS
// through a ring of kSharedStages pairs (LDS DMA; wave w fills K (w even) or V (w odd) of page w / 2
// of the pair), one barrier per pair; per pair a wave forms S^T with 16x16x32 MFMAs, masks the
// columns whose sequence maps the page elsewhere, and adds V^T.P^T with 16x16x32 MFMAs whose 32
// keys are the pair's (keys 4 grp .. +3 of either page per lane group, as the scores lie).  Waves
// keep their own columns, so nothing is merged.  HBM-bound: each page is read once for up to 192
// (head_dim 256: 128) query columns.  32 sequences of 16385 .. 17473 tokens on one 16384-token
// prefix, 40 query heads over 8 of head_dim 128: 167 -> 41 us, its merge of 32 ranges 4.8 -> 10.4;
// 16 sequences of 8000 .. 8192 on one prefix, 16 heads over 8 of head_dim 256, transposed V, capped:
// 184 -> 58 us a call.
template <int D, bool VT, bool CAP>
__device__ __forceinline__ void shared_pages(const DecodeArgs &a, const GroupState &gs, int lane_full,
                                             int hg, int p_lo, int n_range, int slot, char *smem,
                                             int32_t *pgs, uint32_t *msk, const int32_t *ranks) {
  constexpr int NCB = shared_blocks(D);
  constexpr int KS = D / 32, DT = D / 16, KCH = D / 8;
  constexpr int ROWB = 2 * D;
  constexpr int PAGEB = 16 * ROWB;              // bytes of a page's K or V of one head
  constexpr int STAGEB = 4 * PAGEB;             // K, V of page 0, K, V of page 1
  constexpr int NI = PAGEB / 1024;              // DMA instructions per wave and pair
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  const int h = hg / a.n_qgroups, g_lo = hg % a.n_qgroups * 16;
  const int g_cnt = min(16, a.group - g_lo);
  const int per_block = a.group >= 16 ? 1 : 16 / a.group;
  const int n_blocks = (gs.n_sh + per_block - 1) / per_block;
  // row of query column qn of column block cb: head g_lo + qn % g_cnt of sharer
  // cb * per_block + qn / g_cnt; -1: none
  const int in_block = qn / g_cnt;
  auto seq_of = [&](int cb) {
    const int r = cb * per_block + in_block;
    return in_block < per_block && r < gs.n_sh ? ranks[r] : -1;
  };
  auto row_of = [&](int cb) {
    const int j = seq_of(cb);
    return j < 0 ? -1 : (gs.b0 + j) * a.n_q_heads + h * a.group + g_lo + qn - in_block * g_cnt;
  };

  // ---- the range's physical pages and, per page, the sequences that share it: lane = page, wave w
  // takes sequences 8 w .. 8 w + 7 (byte w of the page's mask)
  {
    const int32_t *rep = a.maps + (size_t)(gs.b0 + gs.rep) * a.map_stride + p_lo;
    for (int i0 = 0; i0 < n_range; i0 += 64) {
      const int i = i0 + lane, ic = min(i, n_range - 1);
      const int32_t phys = rep[ic];
      int32_t x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[e] = a.maps[(size_t)(gs.b0 + min(8 * wave + e, gs.n - 1)) * a.map_stride + p_lo + ic];
      uint32_t m = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int full = __builtin_amdgcn_readlane(lane_full, 8 * wave + e);
        if ((gs.sharers >> (8 * wave + e) & 1) && p_lo + i < full && x[e] == phys) m |= 1u << e;
      }
      if (i < n_range) {
        if (wave == 0) pgs[i] = phys;
        reinterpret_cast<uint8_t *>(msk)[4 * i + wave] = (uint8_t)m;
      }
    }
  }
  // ---- the list: pages of all the sharers, then those that two or more of them map
  int n_all = 0, n_pages = 0;
  {
    constexpr int NU = kMaxSharedPages / 256;
    int32_t phys[NU];
    uint32_t mask[NU];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = min(tid + 256 * u, n_range - 1);
      phys[u] = pgs[i];
      mask[u] = msk[i];
    }
#pragma unroll
    for (int some = 0; some < 2; ++some) {
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (256 * u >= n_range) break;
        const bool take = tid + 256 * u < n_range && __popc(mask[u]) >= 2 &&
                          (mask[u] != gs.sharers) == some;
        const int i = place(take, n_pages, reinterpret_cast<int32_t *>(smem));   // ends in a barrier
        if (take) {
          pgs[i] = phys[u];
          msk[i] = mask[u];
        }
      }
      if (!some) n_all = n_pages;
    }
  }
  if (n_pages == 0) {
    for (int cb = wave; cb < n_blocks; cb += kDecWaves) store_empty(a, row_of(cb), slot, grp);
    return;
  }
  // ---- queries of this wave's column blocks wave, wave + 4, ...: B operands
  u32x4 qreg[NCB][KS];
  uint32_t bit[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) {
    const int cb = wave + kDecWaves * c;
    const int row = cb < n_blocks ? row_of(cb) : -1;
    bit[c] = row >= 0 ? 1u << seq_of(cb) : 0u;
    const uint16_t *qrow = reinterpret_cast<const uint16_t *>(a.q) + (size_t)max(row, 0) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      qreg[c][s] = row >= 0 ? *reinterpret_cast<const u32x4 *>(qrow + 32 * s + 8 * grp)
                            : u32x4{0u, 0u, 0u, 0u};
  }
  const int my_blocks = n_blocks > wave ? (n_blocks - wave + kDecWaves - 1) / kDecWaves : 0;

  // ---- DMA: instruction i of a wave covers bytes 1024 i + 16 lane of its K or V page in LDS; the
  // source chunk is chosen so that K chunk c of row r sits at c ^ (r & 15) (& 7 for head_dim 64),
  // V chunk c of row r at c ^ vswz(r), transposed V rows (32 bytes a feature) as they are
  const bool is_v = wave & 1;
  const char *src = reinterpret_cast<const char *>(is_v ? a.vc : a.kc);
  uint64_t page_stride = (uint64_t)a.n_kv_heads * PAGEB;
  src += VT && is_v ? (uint64_t)h * D * a.n_cols * 2 : (uint64_t)h * PAGEB;
  if (VT && is_v) page_stride = 32;
  uint32_t voff[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int byte = 1024 * i + 16 * lane;
    if (VT && is_v) {
      voff[i] = (uint32_t)(byte >> 5) * a.n_cols * 2u + (byte & 16);
    } else {
      const int r = byte / ROWB, c = (byte % ROWB) >> 4;
      voff[i] = r * ROWB + 16 * (c ^ (is_v ? vswz<D>(r) : (r & (KCH < 16 ? KCH - 1 : 15))));
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem + (wave >> 1) * 2 * PAGEB + (wave & 1) * PAGEB;
  const int n_pairs = (n_pages + 1) >> 1;
  wait_vm<0>();      // the DMA loads are counted alone
  __syncthreads();   // pgs, msk
  // every step issues one pair (past the end the last page again, unused), so that the counts of
  // loads in flight are the same throughout
  auto issue = [&](int i) {
    const int e = min(2 * i + (wave >> 1), n_pages - 1);
    const uint64_t phys = (uint32_t)__builtin_amdgcn_readfirstlane(pgs[e]);
    const char *ps = src + phys * page_stride;
    const uint32_t dst = lds0 + (i & (kSharedStages - 1)) * STAGEB;
#pragma unroll
    for (int n = 0; n < NI; ++n) dma_s<0>(dst + 1024 * n, ps, voff[n]);
  };

  f32x4 o[NCB][DT];
  float m_ref[NCB], lsum[NCB];
#pragma unroll
  for (int c = 0; c < NCB; ++c) {
#pragma unroll
    for (int t = 0; t < DT; ++t) o[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_ref[c] = -INFINITY;
    lsum[c] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < kSharedStages - 1; ++i) issue(i);
  // One pair.  EACH: some sharer maps a page of it elsewhere.  Its columns' scores of that
  // page become -inf, and its outputs keep away from the page's values, because a probability of 0
  // does not keep out an infinity or a NaN among them (0 x inf): such pairs are taken a page at a time
  // (16 keys) into fresh accumulators, added to the columns that map the page.
  auto pair = [&](int i, auto each) {
    constexpr bool EACH = decltype(each)::value;
    wait_vm<NI *(kSharedStages - 2)>();   // this wave's part of pair i has landed
    tile_barrier();                       // all parts have, and the slot filled next is read out
    issue(i + kSharedStages - 1);
    if (my_blocks == 0) return;
    const char *kt = smem + (i & (kSharedStages - 1)) * STAGEB;
    const char *vt = kt + PAGEB;
    uint32_t mask0 = 0, mask1 = 0;
    if constexpr (EACH) {
      mask0 = msk[2 * i];
      mask1 = 2 * i + 1 < n_pages ? msk[2 * i + 1] : 0u;
    }
    f32x4 s[NCB][2];
#pragma unroll
    for (int c = 0; c < NCB; ++c)
#pragma unroll
      for (int pp = 0; pp < 2; ++pp) s[c][pp] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int pp = 0; pp < 2; ++pp) {
        const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(
            kt + 2 * pp * PAGEB + qn * ROWB +
            16 * ((4 * st + grp) ^ (qn & (KCH < 16 ? KCH - 1 : 15))));
#pragma unroll
        for (int c = 0; c < NCB; ++c)
          s[c][pp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              ka, __builtin_bit_cast(bf16x8, qreg[c][st]), s[c][pp], 0, 0, 0);
      }
    u32x4 pb[NCB];
#pragma unroll
    for (int c = 0; c < NCB; ++c) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float r = s[c][e >> 2][e & 3];
        const float v = CAP ? a.cap_out * tanh_fast(r * a.cap_in) : r * a.scale_log2;
        x[e] = !EACH || ((e < 4 ? mask0 : mask1) & bit[c]) ? v : -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                       fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
      mx = max_x32(max_x16(mx));
      const bool need = mx > m_ref[c] + kDecSlack;
      if (__builtin_amdgcn_ballot_w64(need)) {
        const float nm = need ? mx : m_ref[c];
        // a column that has seen no key yet keeps reference -inf: nothing to rescale
        const float alpha = nm > -INFINITY ? fast_exp2(m_ref[c] - nm) : 0.f;
#pragma unroll
        for (int t = 0; t < DT; ++t) o[c][t] *= alpha;
        lsum[c] *= alpha;
        m_ref[c] = nm;
      }
      const float nm = m_ref[c] > -INFINITY ? m_ref[c] : 0.f;
      uint32_t w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[e] = pack_bf16x2(fast_exp2(x[2 * e] - nm), fast_exp2(x[2 * e + 1] - nm));
        lsum[c] += __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xFFFF0000u);
      }
      pb[c] = u32x4{w[0], w[1], w[2], w[3]};
    }
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      bf16x8 va;
      if constexpr (VT) {
        const char *p0 = vt + (16 * t + qn) * 32 + 8 * grp;
        const u32x2 lo = *reinterpret_cast<const u32x2 *>(p0);
        const u32x2 hi = *reinterpret_cast<const u32x2 *>(p0 + 2 * PAGEB);
        va = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
      } else {
        const int r = 4 * grp + (qn >> 2);
        const int c = 2 * t + ((qn & 3) >> 1);
        const char *p0 = vt + r * ROWB + 16 * (c ^ vswz<D>(r)) + 8 * (qn & 1);
        va = tr_read_pair(p0, p0 + 2 * PAGEB);
      }
#pragma unroll
      for (int c = 0; c < NCB; ++c) {
        if constexpr (!EACH) {
          o[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, __builtin_bit_cast(bf16x8, pb[c]),
                                                            o[c][t], 0, 0, 0);
        } else {
          const u32x4 v = __builtin_bit_cast(u32x4, va);
#pragma unroll
          for (int pp = 0; pp < 2; ++pp) {
            const f32x4 x = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                __builtin_bit_cast(s16x4, u32x2{v[2 * pp], v[2 * pp + 1]}),
                __builtin_bit_cast(s16x4, u32x2{pb[c][2 * pp], pb[c][2 * pp + 1]}),
                f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            const bool in = (pp ? mask1 : mask0) & bit[c];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[c][t][e] += in ? x[e] : 0.f;
          }
        }
      }
    }
  };
  int i = 0;
  for (; i < n_all >> 1; ++i) pair(i, std::false_type{});
  for (; i < n_pairs; ++i) pair(i, std::true_type{});
  wait_vm<0>();      // no DMA may land once the ring is used for something else
#pragma unroll
  for (int c = 0; c < NCB; ++c) {
    const int cb = wave + kDecWaves * c;
    if (cb < n_blocks)
      store_part<D>(a, row_of(cb), slot, o[c], m_ref[c], sum_x32(sum_x16(lsum[c])), grp);
  }
}

// List of the physical pages >= 0 that `pick` gives for pages [p_lo, p_hi), in page order; returns its
// length.  Called by the whole workgroup.
template <typename F>
__device__ __forceinline__ int build_list(int p_lo, int p_hi, int32_t *pgs, int32_t *wave_cnt, F pick) {
  int n = 0;
  for (int base = p_lo; base < p_hi; base += 256) {
    const int p = base + threadIdx.x;
    const int32_t phys = p < p_hi ? pick(p) : -1;
    const int i = place(phys >= 0, n, wave_cnt);
    if (phys >= 0) pgs[i] = phys;
  }
  __syncthreads();
  return n;
}

// SH: the launch looks for pages that sequences share (shared_pages); a workgroup of a sharer first takes
// a range of them, if there is one for it, then the rest of its own split's pages.
template <int D, bool VT, bool CAP, bool SH>
__device__ __forceinline__ void decode_bf16(const DecodeArgs &a) {
  constexpr int NP = D == 256 ? 1 : 2;   // pages per step of a wave
  constexpr int KS = D / 32;          // S^T MFMA steps
  constexpr int DT = D / 16;          // O^T tiles
  constexpr int ROWB = 2 * D;         // bytes per key row
  constexpr int VL = VT ? 1 : D / 32; // 16-byte V loads per lane per row-major page
  constexpr int MO_LD = D + 4;        // padded row of the merge buffer (floats)
  constexpr int STAGE_BYTES = VT ? 0 : kDecWaves * NP * 16 * ROWB;
  constexpr int MERGE_BYTES = 2 * 16 * MO_LD * 4 + 2 * 2 * 16 * 4;
  constexpr int OWN_BYTES = STAGE_BYTES > MERGE_BYTES ? STAGE_BYTES : MERGE_BYTES;
  constexpr int RING_BYTES = SH ? kSharedStages * 64 * ROWB : 0;
  constexpr int SMEM = OWN_BYTES > RING_BYTES ? OWN_BYTES : RING_BYTES;
  __shared__ __align__(1024) char smem[SMEM];
  __shared__ int32_t pgs[kMaxSplitPages];
  __shared__ uint32_t msk[SH ? kMaxSharedPages : 1];   // sharers of each page of a range
  __shared__ int32_t ranks[SH ? kMaxGroupSeqs : 1];    // the sharers, as indices in the group

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 15, grp = lane >> 4;
  int b, hg, split, len;
  int full = 0;            // lanes j, j + 32: whole pages of sequence j of the group
  bool listed = false;     // the sequence is a sharer: its shared pages leave its own list
  GroupState gs{};
  if constexpr (SH) {
    // KV heads vary fastest, so an XCD keeps its heads, then groups.  Within a group that shares pages
    // splits vary slowest: the ranges, which the first ids have, go with the splits that lose their
    // pages to them, and every CU gets workgroups of both kinds (all of 16384 tokens shared 58 -> 54 us,
    // half of them 270 -> 244); so it is where most sequences are half as long as the bound or less and
    // leave their later splits empty (32 of 4096 tokens in a launch for 17473: 125 -> 100).  Else sequences
    // do: two sequences' workgroups for one split meet on a CU, and in its L1 where they read the same
    // pages after all (31 of 32 sequences on a prefix that the first does not have: 184 -> 170).
    const int n_hq = a.n_kv_heads * a.n_qgroups;
    hg = blockIdx.x % n_hq;
    hg = hg % a.n_kv_heads * a.n_qgroups + hg / a.n_kv_heads;
    // (the last group may be smaller: its workgroups end first)
    int xg = blockIdx.x / n_hq;
    const int n_last = (a.n_seqs - (a.n_groups - 1) * a.group_seqs) * a.own_splits;
    const int n_side = xg < n_last * a.n_groups ? a.n_groups : a.n_groups - 1;
    if (n_side < a.n_groups) xg -= n_last * a.n_groups;
    const int g = xg % n_side;
    xg = xg / n_side + (n_side < a.n_groups ? n_last : 0);
    const int lb = min(g * a.group_seqs + min(lane & 31, a.group_seqs - 1), a.n_seqs - 1);
    const int lane_len = seq_len_of(a, lb);
    const int32_t page = a.maps[(size_t)lb * a.map_stride + a.share_pages / 2];
    full = lane_len >> 4;
    gs = group_state(a, g, full, page);
    split = gs.by_split ? xg / gs.n : xg % a.own_splits;
    b = gs.b0 + (gs.by_split ? xg % gs.n : xg / a.own_splits);
    len = __builtin_amdgcn_readlane(lane_len, b - gs.b0);
    listed = gs.sharers >> (b - gs.b0) & 1;
    int n_ranges = 0, range_pages = 0;
    if (listed) shared_ranges(a, gs, n_ranges, range_pages);
    if (split == 0 && hg == 0 && tid == 0) a.flags[b] = n_ranges;
    if (listed) {
      if (lane < 32 && (gs.sharers >> lane & 1)) ranks[__popc(gs.sharers & ((1u << lane) - 1))] = lane;
      // the sharers' first splits come first: it is they that lose their pages to the ranges
      const int range = split * gs.n_sh + __popc(gs.sharers & ((1u << (b - gs.b0)) - 1));
      if (range < n_ranges) {
        const int p_lo = range * range_pages;
        shared_pages<D, VT, CAP>(a, gs, full, hg, p_lo, min(range_pages, gs.rep_full - p_lo),
                                 a.own_splits + range, smem, pgs, msk, ranks);
      }
      __syncthreads();   // ranks; the lists and the ring are used again
    }
  } else {
    split = blockIdx.x;
    hg = blockIdx.y;
    b = blockIdx.z;
    len = seq_len_of(a, b);
  }
  const int qg = hg % a.n_qgroups;
  const int h = hg / a.n_qgroups;
  const int g_lo = qg * 16;
  const int g_cnt = min(16, a.group - g_lo);     // query heads of this workgroup
  const int hq0 = h * a.group + g_lo;            // first of them
  uint16_t *out = reinterpret_cast<uint16_t *>(a.out);

  if (len == 0) {
    if (split == 0)
      for (int i = tid; i < g_cnt * D; i += 256)
        out[((size_t)b * a.n_q_heads + hq0) * D + i] = 0;
    return;
  }
  const int n_pages = (len + 15) >> 4;
  const int p_begin = split * a.split_pages;
  if (p_begin >= n_pages) return;
  const int p_end = min(p_begin + a.split_pages, n_pages);
  const int n_splits = (n_pages + a.split_pages - 1) / a.split_pages;

  // ---- queries: B operand of S^T = K.Q^T, column qn = query head hq0 + qn
  const bool q_ok = qn < g_cnt;
  u32x4 qreg[KS];
  {
    const uint16_t *qrow =
        reinterpret_cast<const uint16_t *>(a.q) + ((size_t)b * a.n_q_heads + hq0 + qn) * D;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      qreg[s] = q_ok ? *reinterpret_cast<const u32x4 *>(qrow + 32 * s + 8 * grp)
                     : u32x4{0u, 0u, 0u, 0u};
  }

  // the split's physical pages, staged in LDS once (those that its group shares are left out)
  int n_sp = p_end - p_begin;
  const int32_t *map = a.maps + (size_t)b * a.map_stride;
  if (listed) {
    const int32_t *rep = a.maps + (size_t)(gs.b0 + gs.rep) * a.map_stride;
    const int n_shared = min(len >> 4, gs.rep_full);
    n_sp = build_list(p_begin, p_end, pgs, reinterpret_cast<int32_t *>(smem), [&](int p) {
      const int32_t mine = map[p];
      if (b != gs.b0 + gs.rep) return mine == rep[p] && p < n_shared ? -1 : mine;
      // the representative (the first sharer): does another one map its page?
      bool found = false;
      for (int r0 = 1; r0 < gs.n_sh && __builtin_amdgcn_ballot_w64(!found && p < n_shared); r0 += 8) {
        int32_t x[8], j[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          j[e] = __builtin_amdgcn_readfirstlane(ranks[min(r0 + e, gs.n_sh - 1)]);
          x[e] = a.maps[(size_t)(gs.b0 + j[e]) * a.map_stride + p];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          found |= p < __builtin_amdgcn_readlane(full, j[e]) && x[e] == mine;
      }
      return found && p < n_shared ? -1 : mine;
    });
    if (n_sp == 0) {
      if (wave == 0 && qn < g_cnt) store_empty(a, b * a.n_q_heads + hq0 + qn, split, grp);
      return;
    }
  } else {
    for (int i = tid; i < n_sp; i += 256) pgs[i] = map[p_begin + i];
    __syncthreads();
  }
  // keys of entry i of the list: all but the sequence's last page, which no sequence shares unless it is
  // whole, are whole pages
  const int last_keys = p_end == n_pages ? len - 16 * (n_pages - 1) : 16;
  auto keys_of = [&](int i) { return i == n_sp - 1 ? last_keys : 16; };
  const uint32_t page_elems = (uint32_t)a.n_kv_heads * 16u * D;
  const char *kbase = reinterpret_cast<const char *>(a.kc) + (size_t)h * 16 * ROWB;
  const char *vbase = VT ? reinterpret_cast<const char *>(a.vc) + (size_t)h * D * a.n_cols * 2
                         : reinterpret_cast<const char *>(a.vc) + (size_t)h * 16 * ROWB;
  char *vstage = smem + wave * NP * 16 * ROWB;

  struct Page {
    u32x4 k[KS];
    u32x4 v[VT ? 1 : VL];
    u32x2 vt[VT ? DT : 1];
  };

  // A page of nvalid keys.  Loads only; the last page's masking happens in compute_pair, so that no
  // load result is needed here.
  auto load_page = [&](int nvalid, uint32_t phys, Page &pg) {
    const char *kp = kbase + (size_t)phys * page_elems * 2;
    const int krow = min(qn, nvalid - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s)
      pg.k[s] = *reinterpret_cast<const u32x4 *>(kp + krow * ROWB + 64 * s + 16 * grp);
    if constexpr (!VT) {
      const char *vp = vbase + (size_t)phys * page_elems * 2;
#pragma unroll
      for (int j = 0; j < VL; ++j) {
        const int byte = 16 * lane + 1024 * j;
        const int row = min(byte / ROWB, nvalid - 1);
        pg.v[j] = *reinterpret_cast<const u32x4 *>(vp + row * ROWB + byte % ROWB);
      }
    } else {
      const char *vp = vbase + ((size_t)phys * 16 + 4 * grp) * 2;
#pragma unroll
      for (int t = 0; t < DT; ++t)
        pg.vt[t] = *reinterpret_cast<const u32x2 *>(vp + (size_t)(16 * t + qn) * a.n_cols * 2);
    }
  };

  f32x4 o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_ref = -INFINITY;   // reference of query column qn (equal across the 4 lane groups)
  float lsum = 0.f;          // sum of this lane's rounded probabilities

  // Two pages at a time: 32 keys are the k extent of the 16x16x32 MFMA, lane group grp holding keys
  // 4 grp .. +3 of either page, and one softmax step serves both.  (head_dim 256: one page, whose
  // two register buffers are as large.)
  struct Pair {
    Page pg[NP];
  };
  auto compute_pair = [&](const int (&keys)[NP], bool two, const Pair &pr) {
    float x[4 * NP];
#pragma unroll
    for (int pp = 0; pp < NP; ++pp) {
      f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < KS; ++st)
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, pr.pg[pp].k[st]),
                                                    __builtin_bit_cast(bf16x8, qreg[st]), s, 0, 0,
                                                    0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = CAP ? a.cap_out * tanh_fast(s[i] * a.cap_in) : s[i] * a.scale_log2;
        x[4 * pp + i] = 4 * grp + i < keys[pp] && (pp == 0 || two) ? v : -INFINITY;
      }
    }
    float mx = x[0];
#pragma unroll
    for (int e = 1; e < 4 * NP; ++e) mx = fmaxf(mx, x[e]);
    mx = max_x32(max_x16(mx));
    const bool need = mx > m_ref + kDecSlack;
    if (__builtin_amdgcn_ballot_w64(need)) {
      const float nm = need ? mx : m_ref;
      const float alpha = fast_exp2(m_ref - nm);
#pragma unroll
      for (int t = 0; t < DT; ++t) o[t] *= alpha;
      lsum *= alpha;
      m_ref = nm;
    }
    uint32_t w[2 * NP];
#pragma unroll
    for (int e = 0; e < 2 * NP; ++e) {
      w[e] = pack_bf16x2(fast_exp2(x[2 * e] - m_ref), fast_exp2(x[2 * e + 1] - m_ref));
      lsum += __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xFFFF0000u);
    }
    // O^T tile += V^T.P^T with the lane's V of each page, 4 keys of one feature
    auto pv = [&](f32x4 &acc, const u32x2 (&v)[NP]) {
      if constexpr (NP == 2)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, u32x4{v[0][0], v[0][1], v[NP - 1][0], v[NP - 1][1]}),
            __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2 * NP - 2], w[2 * NP - 1]}), acc, 0, 0,
            0);
      else
        acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, v[0]),
                                                        __builtin_bit_cast(s16x4, u32x2{w[0], w[1]}),
                                                        acc, 0, 0, 0);
    };
    // (a page alone: the values beside it are zeros, for 0 x inf is NaN)
    if constexpr (!VT) {
#pragma unroll
      for (int pp = 0; pp < NP; ++pp)
#pragma unroll
        for (int j = 0; j < VL; ++j) {
          const int byte = 16 * lane + 1024 * j;
          const int row = byte / ROWB, c = (byte % ROWB) >> 4;
          *reinterpret_cast<u32x4 *>(vstage + pp * 16 * ROWB + row * ROWB +
                                     16 * (c ^ vswz<D>(row))) =
              pp == 0 || two ? pr.pg[pp].v[j] : u32x4{0u, 0u, 0u, 0u};
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int r = 4 * grp + (qn >> 2);
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const int c = 2 * t + ((qn & 3) >> 1);
        const char *src = vstage + r * ROWB + 16 * (c ^ vswz<D>(r)) + 8 * (qn & 1);
        u32x2 v[NP];
#pragma unroll
        for (int pp = 0; pp < NP; ++pp)
          v[pp] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                (lds_s16x4 *)(src + pp * 16 * ROWB)));
        pv(o[t], v);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      // slots past the sequence end may hold anything: zero this lane's keys beyond it
      u32x2 m[NP];
#pragma unroll
      for (int pp = 0; pp < NP; ++pp) {
        const int keep = pp == 0 || two ? keys[pp] - 4 * grp : 0;
        m[pp][0] = keep >= 2 ? 0xFFFFFFFFu : keep == 1 ? 0x0000FFFFu : 0u;
        m[pp][1] = keep >= 4 ? 0xFFFFFFFFu : keep == 3 ? 0x0000FFFFu : 0u;
      }
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        u32x2 v[NP];
#pragma unroll
        for (int pp = 0; pp < NP; ++pp)
          v[pp] = u32x2{pr.pg[pp].vt[t][0] & m[pp][0], pr.pg[pp].vt[t][1] & m[pp][1]};
        pv(o[t], v);
      }
    }
  };

  // ---- this wave's pairs of list entries wave + 4 k, k = 0 .. n_mine - 1, through two register
  // buffers: a pair is loading while the other is computed.  Every step issues one pair of loads
  // (entries past the list's end re-read its last page, masked or unused), so the wait before each
  // computation leaves the younger pair in flight.
  {
    const int n_pairs = (n_sp + NP - 1) / NP;
    const int n_mine = wave < n_pairs ? (n_pairs - wave + kDecWaves - 1) / kDecWaves : 0;
    if (n_mine > 0) {
      auto entry = [&](int k) { return NP * (wave + kDecWaves * k); };
      auto issue = [&](int k, Pair &pr) {
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) {
          const int e = min(entry(min(k, n_mine - 1)) + pp, n_sp - 1);
          load_page(keys_of(e), (uint32_t)__builtin_amdgcn_readfirstlane(pgs[e]), pr.pg[pp]);
        }
      };
      auto compute = [&](int k, const Pair &pr) {
        const int e = entry(k);
        int keys[NP];
#pragma unroll
        for (int pp = 0; pp < NP; ++pp) keys[pp] = keys_of(min(e + pp, n_sp - 1));
        compute_pair(keys, e + 1 < n_sp, pr);
      };
      Pair b0, b1;
      issue(0, b0);
      // The scheduling barriers keep a pair's loads ahead of the other pair's computation, which the
      // scheduler would otherwise start first, to reuse its registers as they are read; one loop
      // exit, because a second one is routed through a block that also leads back into the loop,
      // and the waits for loads then count that path too.
      int k = 0;
      for (; k + 1 < n_mine; k += 2) {
        issue(k + 1, b1);
        __builtin_amdgcn_sched_barrier(0);
        compute(k, b0);
        __builtin_amdgcn_sched_barrier(0);
        issue(k + 2, b0);
        __builtin_amdgcn_sched_barrier(0);
        compute(k + 1, b1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (k < n_mine) compute(k, b0);
    }
  }

  // ---- merge the 4 waves' (m, l, O^T) in registers, pairwise through LDS: waves 2 and 3 into
  // waves 0 and 1, then wave 1 into wave 0, which writes the result
  lsum = sum_x32(sum_x16(lsum));
  float *mo = reinterpret_cast<float *>(smem);   // [2 slots][16 columns][MO_LD]
  float *mml = mo + 2 * 16 * MO_LD;              // [2 slots][16 columns][m, l]
  auto store_state = [&](int slot) {
#pragma unroll
    for (int t = 0; t < DT; ++t)
      *reinterpret_cast<f32x4 *>(mo + (slot * 16 + qn) * MO_LD + 16 * t + 4 * grp) = o[t];
    if (grp == 0) {
      mml[2 * (slot * 16 + qn)] = m_ref;
      mml[2 * (slot * 16 + qn) + 1] = lsum;
    }
  };
  auto merge_state = [&](int slot) {
    const float mb = mml[2 * (slot * 16 + qn)];
    const float lb = mml[2 * (slot * 16 + qn) + 1];
    const float M = fmaxf(m_ref, mb);
    // a wave that saw no page has m = -inf and contributes nothing
    const float wa = m_ref > -INFINITY ? fast_exp2(m_ref - M) : 0.f;
    const float wb = mb > -INFINITY ? fast_exp2(mb - M) : 0.f;
#pragma unroll
    for (int t = 0; t < DT; ++t) {
      const f32x4 ob =
          *reinterpret_cast<const f32x4 *>(mo + (slot * 16 + qn) * MO_LD + 16 * t + 4 * grp);
      o[t] = o[t] * wa + ob * wb;
    }
    lsum = lsum * wa + lb * wb;
    m_ref = M;
  };
  __syncthreads();   // the V staging slots are reused
  if (wave >= 2) store_state(wave - 2);
  __syncthreads();
  if (wave < 2) merge_state(wave);
  __syncthreads();
  if (wave == 1) store_state(0);
  __syncthreads();
  if (wave != 0) return;
  merge_state(0);
  if (!q_ok) return;
  const int row = b * a.n_q_heads + hq0 + qn;
  if (n_splits == 1 && !listed) {
    const float inv = 1.0f / lsum;
#pragma unroll
    for (int t = 0; t < DT; ++t)
      *reinterpret_cast<u32x2 *>(out + (size_t)row * D + 16 * t + 4 * grp) =
          u32x2{pack_bf16x2(o[t][0] * inv, o[t][1] * inv),
                pack_bf16x2(o[t][2] * inv, o[t][3] * inv)};
  } else {
    store_part<D>(a, row, split, o, m_ref, lsum, grp);
  }
}

template <int D, bool VT, bool CAP>
__global__ __launch_bounds__(256, D == 64 ? 3 : D == 128 ? 2 : 1) void decode_bf16_kernel(DecodeArgs a) {
  decode_bf16<D, VT, CAP, false>(a);
}
template <int D, bool VT, bool CAP>
__global__ __launch_bounds__(256, D < 256 ? 2 : 1) void decode_bf16_shared_kernel(DecodeArgs a) {
  decode_bf16<D, VT, CAP, true>(a);
}

// fp32 caches: one wave per (sequence, query head, split), VALU dot products.  Lane l holds key
// l % 16 of a page and a quarter of its features; the quarters are summed across lanes.
template <bool VT, bool CAP>
__global__ __launch_bounds__(64) void decode_f32_kernel(DecodeArgs a, int D) {
  const int lane = threadIdx.x;
  const int kq = lane & 15, quarter = lane >> 4;
  const int b = blockIdx.z, hq = blockIdx.y, split = blockIdx.x;
  const int h = hq / a.group;
  float *out = reinterpret_cast<float *>(a.out);
  const int len = seq_len_of(a, b);
  const size_t row = (size_t)b * a.n_q_heads + hq;
  if (len == 0) {
    if (split == 0)
      for (int d = lane; d < D; d += 64) out[row * D + d] = 0.f;
    return;
  }
  const int n_pages = (len + 15) >> 4;
  const int p_begin = split * a.split_pages;
  if (p_begin >= n_pages) return;
  const int p_end = min(p_begin + a.split_pages, n_pages);
  const int n_splits = (n_pages + a.split_pages - 1) / a.split_pages;
  const float *q = reinterpret_cast<const float *>(a.q) + row * D;
  const float *kc = reinterpret_cast<const float *>(a.kc);
  const float *vc = reinterpret_cast<const float *>(a.vc);
  const int32_t *map = a.maps + (size_t)b * a.map_stride;
  const int qd = D / 4;                       // features per quarter
  const int dpl = (D + 63) / 64;              // output features per lane (<= 4)
  float o[4] = {0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  for (int p = p_begin; p < p_end; ++p) {
    const uint32_t phys = (uint32_t)map[p];
    const int nvalid = min(16, len - 16 * p);
    const float *kr = kc + (((size_t)phys * a.n_kv_heads + h) * 16 + min(kq, nvalid - 1)) * D;
    float s = 0.f;
    for (int e = 0; e < qd; ++e) s = fmaf(q[quarter * qd + e], kr[quarter * qd + e], s);
    s = sum_x32(sum_x16(s));
    float x = CAP ? a.cap_out * tanh_fast(s * a.cap_in) : s * a.scale_log2;
    if (kq >= nvalid) x = -INFINITY;
    float mx = x;
    for (int off = 1; off < 16; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    const float nm = fmaxf(m_run, mx);
    const float alpha = fast_exp2(m_run - nm);
    m_run = nm;
    const float pk = fast_exp2(x - nm);        // lanes 0..15 hold the page's 16 probabilities
    float ps = pk;
    for (int off = 1; off < 16; off <<= 1) ps += __shfl_xor(ps, off);
    l_run = l_run * alpha + ps;
    for (int j = 0; j < dpl; ++j) o[j] *= alpha;
    for (int k = 0; k < nvalid; ++k) {
      const float pkk = __shfl(pk, k);
      for (int j = 0; j < dpl; ++j) {
        const int d = lane + 64 * j;
        if (d >= D) break;
        const float v = VT ? vc[((size_t)h * D + d) * a.n_cols + phys * 16 + k]
                           : vc[(((size_t)phys * a.n_kv_heads + h) * 16 + k) * D + d];
        o[j] = fmaf(pkk, v, o[j]);
      }
    }
  }
  const size_t slot = row * a.max_splits + split;
  for (int j = 0; j < dpl; ++j) {
    const int d = lane + 64 * j;
    if (d >= D) break;
    if (n_splits == 1) out[row * D + d] = o[j] / l_run;
    else a.part[slot * D + d] = o[j];
  }
  if (n_splits > 1 && lane == 0) {
    a.part_ml[2 * slot] = m_run;
    a.part_ml[2 * slot + 1] = l_run;
  }
}

// Merge of the partials of every (sequence, query head) that has more than one split, or any under
// shared pages: one wave per (sequence, query head).  D / 4 lanes cover a partial row in 16-byte
// loads, so a wave reads 64 / (D / 4) partials per instruction; the first kPre instructions are
// issued with the (m, l) pairs, so that the round trips to memory overlap.  Lane k holds the
// weight of slot 64 c + k; partials are added in order within each of the wave's shares, the
// shares at the end.  A partial with m = -inf holds nothing (no page was left to it) and its
// output is never used.
template <bool BF16>
__global__ __launch_bounds__(64) void decode_combine_kernel(DecodeArgs a, int D, int lpr_shift) {
  constexpr int kPre = 20, kQuad = 4;   // load instructions in flight together; skipped by fours
  const int lane = threadIdx.x;
  const int hq = blockIdx.x, b = blockIdx.y;
  const size_t row = (size_t)b * a.n_q_heads + hq;
  const float2 *ml = reinterpret_cast<const float2 *>(a.part_ml) + row * a.max_splits;
  const float *po = a.part + row * a.max_splits * D;
  const int share = lane >> lpr_shift, n_shares = 64 >> lpr_shift;
  const int d = 4 * (lane & ((1 << lpr_shift) - 1));
  f32x4 pre[kPre];
  auto load = [&](int s0, int end) {
#pragma unroll
    for (int i0 = 0; i0 < kPre; i0 += kQuad) {
      if (s0 + i0 * n_shares >= end) continue;
#pragma unroll
      for (int i = i0; i < i0 + kQuad; ++i) {
        const int s = s0 + i * n_shares + share;
        if (s < end) pre[i] = *reinterpret_cast<const f32x4 *>(po + (size_t)s * D + d);
      }
    }
  };
  // The first loads do not wait for the sequence's length (a slot that turns out to hold nothing
  // is not used), so the launch is one round trip for all but the longest rows.
  load(0, a.own_splits);
  float2 ml0 = lane < a.max_splits ? ml[lane] : float2{-INFINITY, 0.f};
  int shares = 0;                   // the row's partials of shared pages
  if (a.n_groups > 0) shares = a.flags[b];
  const int len = seq_len_of(a, b);
  const int n_pages = (len + 15) >> 4;
  const int n_own = (n_pages + a.split_pages - 1) / a.split_pages;
  if (n_own == 0 || (n_own == 1 && !shares)) return;
  // the row's partials: slots below n_own and, with shared pages, those from own_splits on
  const int ns = shares ? a.own_splits + shares : n_own;
  auto used = [&](int s) { return s < n_own || (s >= a.own_splits && s < ns); };
  if (shares && kPre * n_shares > a.own_splits) {
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int s = i * n_shares + share;
      if (s >= a.own_splits && s < ns)
        pre[i] = *reinterpret_cast<const f32x4 *>(po + (size_t)s * D + d);
    }
  }
  // the first 64 pairs stay in registers, the others (very long sequences) are read again
  if (!used(lane)) ml0 = float2{-INFINITY, 0.f};
  float M = ml0.x;
  for (int s = lane + 64; s < ns; s += 64)
    if (used(s)) M = fmaxf(M, ml[s].x);
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  float lsum = used(lane) ? ml0.y * fast_exp2(ml0.x - M) : 0.f;
  for (int s = lane + 64; s < ns; s += 64)
    if (used(s)) lsum += ml[s].y * fast_exp2(ml[s].x - M);
  for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off);
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  // -1: an empty partial
  auto weight = [&](float m) { return m == -INFINITY ? -1.f : fast_exp2(m - M); };
  float wl = weight(ml0.x);
  int w0 = 0;                       // partial whose weight lane 0 holds
  for (int s0 = 0; s0 < ns; s0 += kPre * n_shares) {
    if (s0 > 0) load(s0, ns);
#pragma unroll
    for (int i0 = 0; i0 < kPre; i0 += kQuad) {
      if (s0 + i0 * n_shares >= ns) continue;
#pragma unroll
      for (int i = i0; i < i0 + kQuad; ++i) {
        const int s1 = s0 + i * n_shares;
        if (s1 < ns && s1 - w0 >= 64) {   // (n_shares divides 64)
          w0 += 64;
          wl = weight(used(w0 + lane) ? ml[w0 + lane].x : -INFINITY);
        }
        const float w = __shfl(wl, (s1 - w0 + share) & 63);
        if (used(s1 + share) && w != -1.f) o += pre[i] * w;
      }
    }
  }
  for (int off = 32; off >= 1 << lpr_shift; off >>= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] += __shfl_xor(o[e], off);
  if (share != 0) return;
  const float inv = 1.0f / lsum;
  if (BF16)
    *reinterpret_cast<u32x2 *>(reinterpret_cast<uint16_t *>(a.out) + row * D + d) =
        u32x2{pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv)};
  else
    *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + row * D + d) = o * inv;
}

}  // namespace

int decode_split_pages(int32_t n_seqs, int32_t n_kv_heads, int32_t wgs_per_kv_head,
                       int32_t max_len) {
  // Measured on MI355X (256 CUs, two of these workgroups resident per CU): about 512
  // workgroups over the longest sequence, at least 32 pages (8 per wave) per split so that a
  // workgroup's set-up is amortised, and no partial second round of workgroups: between 256
  // and 512 workgroups, 256 is faster.
  constexpr int64_t kCUs = 256;
  constexpr int64_t kMinSplitPages = 32;
  const int64_t max_pages = ((int64_t)max_len + 15) / 16;
  if (max_pages <= 0) return 1;
  const int64_t pairs = (int64_t)n_seqs * n_kv_heads * wgs_per_kv_head;
  int64_t ns = (2 * kCUs + pairs - 1) / pairs;
  int64_t sp = (max_pages + ns - 1) / ns;
  if (sp < kMinSplitPages) sp = kMinSplitPages;
  ns = (max_pages + sp - 1) / sp;
  if (pairs * ns > kCUs && pairs * ns < 2 * kCUs && pairs <= kCUs) {
    ns = kCUs / pairs;
    sp = (max_pages + ns - 1) / ns;
  }
  // bounds of the page list in LDS and of the merge loop
  if (sp < (max_pages + kMaxDecSplits - 1) / kMaxDecSplits)
    sp = (max_pages + kMaxDecSplits - 1) / kMaxDecSplits;
  if (sp > kMaxSplitPages) sp = kMaxSplitPages;
  if (sp > max_pages) sp = max_pages;
  return (int)sp;
}

namespace {

// Shape of a launch: splits of each sequence's own pages, and the groups and page ranges of the
// pages that sequences share.
struct DecodeShape {
  int split_pages, own_splits;         // pages per split, splits of the longest sequence
  int n_groups, group_seqs;            // 0 groups: shared pages are not looked for
  int shared_splits;                   // ranges of a group's shared pages at most
  int slots() const { return own_splits + (n_groups ? shared_splits : 0); }
};

// Workspace bytes of `slots` partials a row.
size_t part_bytes(const DecodeLaunch &p, int64_t slots) {
  return (size_t)p.n_seqs * p.n_q_heads * slots * (p.head_dim + 2) * sizeof(float);
}
size_t shape_bytes(const DecodeLaunch &p, const DecodeShape &s) {
  if (s.slots() <= 1) return 0;
  return part_bytes(p, s.slots()) + (s.n_groups ? (size_t)p.n_seqs * sizeof(int32_t) : 0);
}

// The shape that fits a workspace of ws_bytes: the splits of the sequences' own pages always do (the
// call is refused otherwise), shared pages are cut into as many ranges as it holds partials for, and not
// looked for where it holds too few.
DecodeShape decode_shape(const DecodeLaunch &p, size_t ws_bytes) {
  DecodeShape s{};
  const int group = p.n_q_heads / p.n_kv_heads;
  // bf16: one workgroup per 16 query heads of a group; f32: one wave per query head
  const int per_kv = p.is_bf16 ? (group + 15) / 16 : group;
  s.split_pages = decode_split_pages(p.n_seqs, p.n_kv_heads, per_kv, p.max_len);
  const int64_t max_pages = ((int64_t)p.max_len + 15) / 16;
  s.own_splits = (int)((max_pages + s.split_pages - 1) / s.split_pages);
  if (s.own_splits < 1) s.own_splits = 1;
  // Shared pages are looked for where the sequences' keys and values may pass twice the 256 MB last-level
  // cache (below, the caches serve the repeated reads); a launch of one split a sequence, which needs
  // no merge as it is, must gain that too (128 sequences of 1200 tokens, nothing shared: 111 us,
  // looked for 114).  A look costs 1 to 2 us where nothing is shared.
  const int64_t kv_bytes = (int64_t)p.n_seqs * p.max_len * p.n_kv_heads * p.head_dim * 4;
  if (!p.is_bf16 || p.n_seqs < 2 || kv_bytes < (s.own_splits > 1 ? 1 : 4) * kSharedMinBytes) return s;
  // such a launch has its workgroups in one grid dimension, which holds less than 2^32 threads
  if ((int64_t)p.n_kv_heads * per_kv * p.n_seqs * s.own_splits > UINT32_MAX / 256) return s;
  // sequences per group: what the column blocks of a workgroup hold
  const int per_block = group >= 16 ? 1 : 16 / group;
  const int cap = std::min(kMaxGroupSeqs, kDecWaves * shared_blocks(p.head_dim) * per_block);
  const int n_groups = (p.n_seqs + cap - 1) / cap;
  s.group_seqs = (p.n_seqs + n_groups - 1) / n_groups;
  // about one job of shared pages per CU
  const int64_t heads = (int64_t)((p.n_seqs + s.group_seqs - 1) / s.group_seqs) * p.n_kv_heads * per_kv;
  int64_t ns = heads < 256 ? 256 / heads : 1;
  const size_t fixed = part_bytes(p, s.own_splits) + (size_t)p.n_seqs * sizeof(int32_t);
  const int64_t fit = ws_bytes > fixed ? (int64_t)((ws_bytes - fixed) / part_bytes(p, 1)) : 0;
  if (fit * kMaxSharedPages < max_pages) return s;
  ns = std::min(ns, fit);
  int64_t sp = (max_pages + ns - 1) / ns;
  if (sp < kMinRangePages) sp = kMinRangePages;
  if (sp > kMaxSharedPages) sp = kMaxSharedPages;
  s.n_groups = (p.n_seqs + s.group_seqs - 1) / s.group_seqs;
  s.shared_splits = (int)((max_pages + sp - 1) / sp);
  return s;
}

}  // namespace

size_t decode_workspace_bytes(const DecodeLaunch &p) { return shape_bytes(p, decode_shape(p, SIZE_MAX)); }

size_t decode_workspace_min(const DecodeLaunch &p) { return shape_bytes(p, decode_shape(p, 0)); }

hipError_t launch_decode(const DecodeLaunch &p, hipStream_t stream) {
  const int group = p.n_q_heads / p.n_kv_heads;
  const int n_qgroups = (group + 15) / 16;
  DecodeShape sh = decode_shape(p, p.workspace_bytes);
  // shared pages travel by LDS DMA, 16 aligned bytes a lane: a cache that starts elsewhere is read
  // sequence by sequence
  if ((uintptr_t)p.cache_k % 16 != 0 || (uintptr_t)p.cache_v % 16 != 0) sh.n_groups = 0;
  const int slots = sh.slots();
  DecodeArgs a{};
  const size_t esize = p.is_bf16 ? 2 : 4;
  const size_t layer_elems = (size_t)p.n_phys_pages * p.n_kv_heads * 16 * p.head_dim;
  a.q = p.q;
  a.out = p.out;
  a.kc = reinterpret_cast<const char *>(p.cache_k) + (size_t)p.layer * layer_elems * esize;
  a.vc = reinterpret_cast<const char *>(p.cache_v) + (size_t)p.layer * layer_elems * esize;
  a.maps = p.maps;
  a.lens = p.lens;
  float *ws = reinterpret_cast<float *>(p.workspace);
  const size_t part_elems = (size_t)p.n_seqs * p.n_q_heads * slots * p.head_dim;
  a.part = slots > 1 ? ws : nullptr;
  a.part_ml = slots > 1 ? ws + part_elems : nullptr;
  a.flags = reinterpret_cast<int32_t *>(
      ws + part_elems + (size_t)2 * p.n_seqs * p.n_q_heads * slots);
  a.map_stride = p.map_stride;
  a.max_len = p.max_len;
  a.n_q_heads = p.n_q_heads;
  a.n_kv_heads = p.n_kv_heads;
  a.group = group;
  a.n_qgroups = n_qgroups;
  a.split_pages = sh.split_pages;
  a.max_splits = slots;
  a.n_seqs = p.n_seqs;
  a.n_groups = sh.n_groups;
  a.group_seqs = sh.group_seqs;
  a.shared_splits = sh.shared_splits;
  const int64_t page_bytes = (int64_t)p.n_kv_heads * p.head_dim * 64;
  a.share_pages = (int32_t)(kSharedMinBytes / 2 / page_bytes / p.n_seqs) + 1;
  a.own_splits = sh.own_splits;
  a.n_cols = (uint32_t)p.n_phys_pages * 16u;
  const float log2e = 1.4426950408889634f;
  a.scale_log2 = p.scale * log2e;
  a.cap_in = p.softcap > 0.f ? p.scale / p.softcap : 0.f;
  a.cap_out = p.softcap * log2e;
  const bool cap = p.softcap > 0.f;
  if (p.is_bf16) {
    const int n_hq = p.n_kv_heads * n_qgroups;
    const bool shared = sh.n_groups > 0;
    const dim3 grid =
        shared ? dim3((uint32_t)n_hq * p.n_seqs * sh.own_splits)
               : dim3(sh.own_splits, n_hq, p.n_seqs);
#define NEXUS_DEC(D_, VT_, CAP_)                                                                   \
  do {                                                                                             \
    if (shared)                                                                                    \
      hipLaunchKernelGGL((decode_bf16_shared_kernel<D_, VT_, CAP_>), grid, dim3(256), 0, stream, a); \
    else                                                                                           \
      hipLaunchKernelGGL((decode_bf16_kernel<D_, VT_, CAP_>), grid, dim3(256), 0, stream, a); \
  } while (0)
#define NEXUS_DEC_D(D_)                                             \
  do {                                                              \
    if (p.v_transposed) {                                           \
      if (cap) NEXUS_DEC(D_, true, true); else NEXUS_DEC(D_, true, false);   \
    } else {                                                        \
      if (cap) NEXUS_DEC(D_, false, true); else NEXUS_DEC(D_, false, false); \
    }                                                               \
  } while (0)
    if (p.head_dim == 64) NEXUS_DEC_D(64);
    else if (p.head_dim == 128) NEXUS_DEC_D(128);
    else NEXUS_DEC_D(256);
#undef NEXUS_DEC_D
#undef NEXUS_DEC
  } else {
    const dim3 grid(sh.own_splits, p.n_q_heads, p.n_seqs);
    if (p.v_transposed) {
      if (cap) hipLaunchKernelGGL((decode_f32_kernel<true, true>), grid, dim3(64), 0, stream, a, p.head_dim);
      else hipLaunchKernelGGL((decode_f32_kernel<true, false>), grid, dim3(64), 0, stream, a, p.head_dim);
    } else {
      if (cap) hipLaunchKernelGGL((decode_f32_kernel<false, true>), grid, dim3(64), 0, stream, a, p.head_dim);
      else hipLaunchKernelGGL((decode_f32_kernel<false, false>), grid, dim3(64), 0, stream, a, p.head_dim);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || slots <= 1) return e;
  const dim3 cgrid(p.n_q_heads, p.n_seqs);
  int lpr_shift = 0;                  // log2 of the lanes that cover a partial row
  while ((4 << lpr_shift) < p.head_dim) ++lpr_shift;
  if (p.is_bf16)
    hipLaunchKernelGGL((decode_combine_kernel<true>), cgrid, dim3(64), 0, stream, a, p.head_dim,
                       lpr_shift);
  else
    hipLaunchKernelGGL((decode_combine_kernel<false>), cgrid, dim3(64), 0, stream, a, p.head_dim,
                       lpr_shift);
  return hipGetLastError();
}

}  // namespace nexus
