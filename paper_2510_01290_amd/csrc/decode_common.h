// Split-K bookkeeping shared by the decode-attention kernels and the merge kernel.
//
// The context of one (query, kv-head) -- a "head" below -- is worked on by several items; each
// item leaves, per query head of the group, one partial row (acc[D], m, l, two words of padding):
// the unnormalised weighted value sum, the running maximum of the scaled scores in the log2
// domain, and the sum of 2^(score - m).  The merge kernel folds the rows of a head.
//
// How many items a head gets is decided on the device from its page count, identically by every
// kernel of a call: an item per `ppi` pages, at most `per_head` (both chosen by the host); the items
// of a head that is short do not exist (their waves leave at once).  Item j of n takes the same fraction
// [j/n, (j+1)/n) of each of the three per-type lists.
#pragma once
#include "common.h"

// Waves per SIMD the fast kernel of full-attention layers is built for, and the LDS ring of a wave: together they take
// 144 KB of the compute unit's 160.  More waves hide more of each other's latency, a deeper ring keeps more bytes in
// flight; where the line lies is measured: integer formats at head_dim 128 (18 KB: two pairs of 8-bit, three of 4-bit,
// six of 2-bit pages) 16 x 8k tokens 43 us at two waves, 64 at three; head_dim 64 (12 KB: two, four, eight pairs)
// 287 us at three, 328 at four for 128 x 4k..32k tokens; the paper's formats at 128, whose registers fit a third wave and
// whose arithmetic needs it, 132 at three and 137 at two.  The host sizes launches with the same numbers.
__host__ __device__ constexpr int decode_waves_per_simd(int head_dim, bool fp) { return (head_dim == 64 ? 3 : 2) + (fp ? 1 : 0); }
__host__ __device__ constexpr int stream_ring_bytes(int head_dim, bool fp) { return 147456 / (4 * decode_waves_per_simd(head_dim, fp)); }

// Sliding-window layers: waves of a workgroup, pages of each type it scans at a time, its rings and all its LDS (the rings,
// then per type the ids, masks and list positions of the visible pages, then their counts per wave).
constexpr int kWindowWaves = 8, kWindowBlock = 64 * kWindowWaves;
__host__ __device__ constexpr int window_ring_bytes(int head_dim) { return head_dim == 128 ? 14336 : 9216; }
__host__ __device__ constexpr int window_lds_bytes(int head_dim) { return kWindowWaves * window_ring_bytes(head_dim) + 9 * kWindowBlock * 4 + 3 * kWindowWaves * 4; }

namespace thinkv {

struct DecodeArgs {
  const void* q;
  void* out;
  float* lse;
  const int32_t* seq_ids;
  const int32_t* q_pos;
  float* partial;       // [n_rows][G][D + 4]
  int32_t* alloc;       // [B * n_kv_heads][2]: first row and number of rows of each head, written by its item 0
  int layer, B, window, q_dtype, out_dtype;
  int n_rows;           // items, = per_head * B * n_kv_heads
  int per_head;         // the most items a head can have
  int ppi;              // pages per item
  float scale_log2e;    // softmax_scale * log2(e)
  // sparsity statistic (null / 0 on plain attention calls)
  float* stat;          // [B][n_kv_heads][stat_stride] pooled scores, 16 per page in page-list order (types 0, 1, 2)
  int64_t stat_stride;  // floats per (query, kv-head): 16 * max_ctx_pages
  float* sparsity;      // [B]
  int direct;           // 1: every head has a single item and the attention kernel writes out / lse itself
  int waves;            // fast kernel: waves of an item's workgroup (full attention), kv-heads of one (sliding window)
};

constexpr int kMaxRowsPerHead = 1024;

struct ItemLoc {
  int b, hkv;   // the head
  int j, n;     // item j of n
  int row0;     // the head's first partial row
};

// a value that is the same in all lanes but was read by a vector load, as a scalar: what is computed from it stays scalar
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ inline int seq_pages(const thinkv_view& v, int layer, int seq, int* np) {
  const thinkv_config& c = v.cfg;
  int tot = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    np[k] = (seq >= 0 && seq < c.max_seqs) ? uniform(v.n_pages[npages_index(c, seq, layer, k)]) : 0;
    tot += np[k];
  }
  return tot;
}

// Item id -> head, item number, item count, first row.  Item-major: ids [j * heads, (j + 1) * heads) are item j of every
// head (the hardware starts workgroups in id order and a SIMD favours its oldest wave: every head gets workers of every
// age), shifted by j so that the items of a head land on different XCDs (ids go round the XCDs).
__device__ inline ItemLoc locate_item(const thinkv_view& v, const DecodeArgs& a, int id) {
  const thinkv_config& c = v.cfg;
  const int H = c.n_kv_heads, heads = H * a.B;
  ItemLoc it;
  it.j = uniform(id / heads);   // (divisions are vector arithmetic)
  int rest = id - it.j * heads - uniform(it.j % heads);
  if (rest < 0) rest += heads;
  it.b = uniform(rest / H);
  it.hkv = rest - it.b * H;
  int np[3];
  const int tot = seq_pages(v, a.layer, uniform(a.seq_ids[it.b]), np);
  int n = uniform((int)(((int64_t)tot + a.ppi - 1) / a.ppi));
  n = n < 1 ? 1 : (n > a.per_head ? a.per_head : n);
  it.n = n;
  it.row0 = rest * a.per_head;
  return it;
}

constexpr int kRowPad = 4;   // a partial row: acc[D], m, l, two unused words (rows stay 16-byte aligned)

__device__ inline float* partial_row(const DecodeArgs& a, int G, int D, int row, int g) {
  return a.partial + ((int64_t)row * G + g) * (D + kRowPad);
}

}  // namespace thinkv
