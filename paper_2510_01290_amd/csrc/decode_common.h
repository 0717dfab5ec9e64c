// Split-K bookkeeping shared by the decode-attention kernels and the merge kernel.
//
// The context of one (query, kv-head) -- a "head" below -- is worked on by several items; each
// item leaves, per query head of the group, one partial row (acc[D], m, l, two words of padding):
// the unnormalised weighted value sum, the running maximum of the scaled scores in the log2
// domain, and the sum of 2^(score - m).  The merge kernel folds the rows of a head.
//
// How many items a head gets is decided on the device from page counts, identically by every workgroup of a launch.  Either
// (locate_item) from its own: an item per `ppi` pages, at most `per_head` (both chosen by the host); the items
// of a head that is short do not exist (their waves leave at once).  Or (deal_item) from those of the whole batch, so that the
// items fill the machine once.  Item j of n takes the same fraction [j/n, (j+1)/n) of each of the three per-type lists.
#pragma once
#include "common.h"

// Waves per SIMD the fast kernel of full-attention layers is built for, and the LDS ring of a wave: together they take
// 144 KB of the compute unit's 160.  More waves hide more of each other's latency, a deeper ring keeps more bytes in
// flight; where the line lies is measured: integer formats at head_dim 128 (18 KB: two pairs of 8-bit, three of 4-bit,
// six of 2-bit pages) 16 x 8k tokens 43 us at two waves, 64 at three; head_dim 64 (12 KB: two, four, eight pairs)
// 287 us at three, 328 at four for 128 x 4k..32k tokens; the paper's formats at 128, whose registers fit a third wave:
// 16 x 32k of ternary codes 110 us at three and 119 at two, eight heads a group 107 and 115; of 8-bit types, and of all three, no
// difference (171, 130 and 129), in short or odd batches two are better (17 x 16k 89 and 85, 8 x 2k 21.4 and 18.9).  The host
// sizes launches with the same numbers.
__host__ __device__ constexpr int decode_waves_per_simd(int head_dim, bool fp) { return (head_dim == 64 ? 3 : 2) + (fp ? 1 : 0); }
__host__ __device__ constexpr int stream_ring_bytes(int head_dim, bool fp) { return 147456 / (4 * decode_waves_per_simd(head_dim, fp)); }

// LDS of a wave through which the softmax weights of a pair change layout (0: by a matrix product; see Softmax::weights)
__host__ __device__ constexpr int exchange_bytes(int head_dim, int heads, bool fp) {
  return (fp ? head_dim == 128 : head_dim == 64 && heads == 8) ? 2 * 16 * heads * 4 : 0;
}

// Sliding-window layers: waves of a workgroup (as many as a compute unit holds; a page of each type per thread is scanned at a time), entries
// of a type's list of what is visible, a wave's ring, and all LDS (rings, the lists' page ids, with the statistic list positions, and their
// masks, counts per wave).
constexpr int kWindowList = 1024, kCounts = 16;
__host__ __device__ constexpr int window_waves(int head_dim) { return 4 * decode_waves_per_simd(head_dim, false); }
__host__ __device__ constexpr int window_ring_bytes(int head_dim) { return head_dim == 128 ? 14336 : 9216; }
__host__ __device__ constexpr int window_lds_bytes(int head_dim, bool stat) {
  return window_waves(head_dim) * window_ring_bytes(head_dim) + 3 * kWindowList * (stat ? 10 : 6) + 8 * kCounts;
}

// The statistic's sum over the kv-heads in one word (stat_count_kernel): for up to 2^lg heads a count of lg + 1 bits above 63 - lg bits in units
// of 2^-(62 - 2 lg).  A fraction is a binary32 quotient of counts, 24 bits from 2^-31 on, so a whole number of units for up to sixteen heads whatever the
// context, for 32 up to 2^29 tokens and for 64 up to 2^27, whose keys and values no card holds: nothing is lost, and the mean is rounded once.
constexpr int kStatHeads = 64;

// Items dealt over a batch (deal_item): fewest pages a wave is worth.
constexpr int kDealPages = 8;

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
  unsigned long long* stat_sum;   // [B] sum of the kv-heads' fractions, and how many are in it (stat_count_kernel); null: every fraction by itself
  int direct;           // 1: every head has a single item and the attention kernel writes out / lse itself
  int waves;            // fast kernel: waves of a workgroup (full attention), kv-heads of one (sliding window)
  int grid;             // full attention, items dealt by the batch's page counts: workgroups; 0: locate_item
};

constexpr int kMaxRowsPerHead = 1024;

struct ItemLoc {
  int b, hkv;   // the head
  int j, n;     // item j of n
  int row0;     // the head's first partial row
};

// a value that is the same in all lanes but was read by a vector load, as a scalar: what is computed from it stays scalar
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// x / y of scalars, 0 <= x < 2^24 and 0 < y < 2^24, exactly: the quotient by the reciprocal is at most two off.  (The compiler's
// 32-bit division takes thirty instructions and its 64-bit one 130; six of those to find a wave's share of the page lists were
// 1.7 us of every launch.)
__device__ __forceinline__ int quotient(int x, int y) {
  int q = (int)((float)x * __builtin_amdgcn_rcpf((float)y));
#pragma unroll
  for (int again = 0; again < 2; ++again) {
    const int r = x - q * y;
    q += (r >= y ? 1 : 0) - (r < 0 ? 1 : 0);
  }
  return uniform(q);
}
// x * j / n for 0 <= x < 2^24, 0 <= j <= n <= kMaxRowsPerHead
__device__ __forceinline__ int portion(int x, int j, int n) {
  if (n == 1) return j ? x : 0;
  const int each = quotient(x, n);
  return j * each + quotient(j * (x - n * each), n);
}

__device__ inline int seq_pages(const thinkv_view& v, int layer, int seq, int* np) {
  const thinkv_config& c = v.cfg;
  const bool valid = seq >= 0 && seq < c.max_seqs;
  const int32_t* at = v.n_pages + (valid ? npages_index(c, seq, layer, 0) : 0);   // (there is a first sequence)
  int tot = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) np[k] = uniform(at[k]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    np[k] = valid ? np[k] : 0;
    tot += np[k];
  }
  return tot;
}

// Item id -> head, item number, item count, first row.  Item-major: ids [j * heads, (j + 1) * heads) are item j of every
// head (the hardware starts workgroups in id order and a SIMD favours its oldest wave: every head gets workers of every
// age), shifted by j so that the items of a head land on different XCDs (ids go round the XCDs).
__device__ inline ItemLoc locate_head(const thinkv_config& c, const DecodeArgs& a, int id) {   // ... without the item count
  const int H = c.n_kv_heads, heads = H * a.B;
  ItemLoc it;
  int rest = id;
  it.j = 0;
  if (a.per_head > 1) {
    it.j = uniform(id / heads);
    rest = id - it.j * heads - uniform(it.j % heads);
    if (rest < 0) rest += heads;
  }
  it.b = heads < (1 << 24) ? quotient(rest, H) : uniform(rest / H);
  it.hkv = rest - it.b * H;
  it.n = 0;
  it.row0 = rest * a.per_head;
  return it;
}
// the items of a head whose sequence holds `pages`
__device__ inline void count_items(const DecodeArgs& a, int pages, ItemLoc& it) {
  it.n = 1;
  if (a.per_head > 1) {
    const int n = uniform((int)(((uint32_t)pages + (uint32_t)a.ppi - 1u) / (uint32_t)a.ppi));   // (at most 2^26 pages)
    it.n = n < 1 ? 1 : (n > a.per_head ? a.per_head : n);
  }
}
__device__ inline ItemLoc locate_item(const thinkv_view& v, const DecodeArgs& a, int id) {
  ItemLoc it = locate_head(v.cfg, a, id);
  int np[3];
  count_items(a, seq_pages(v, a.layer, uniform(a.seq_ids[it.b]), np), it);
  return it;
}

// Items in proportion to the pages of the batch's sequences (a.grid > 0; at most kDealSeqs queries): a.grid workgroups of kFull
// waves, a compute unit's worth each, and every item at once.  A workgroup works on `sub` items side by side, each by
// kFull / sub of its waves.  With sub = 1 a batch of 17 x 8 heads leaves 120 of 256 compute units idle, and so do the short
// sequences of a batch of uneven lengths; smaller shares pack better, but each pays for a query, a row and a last
// chunk of its own.  So: the first sub whose workgroups have at most 8 % more pages than they would with everything
// spread evenly, or else the best one, with as many items for the longest sequence as let all items fit and, for the
// others, an item per as many pages.  Every wave works this out for itself, a sequence per lane (under a microsecond, most of
// it loads that it needs in any case).  Measured against items of equal size by the host's bound alone, 8 kv-heads of 128,
// us: 17 x 32k tokens 181, now 139; 20 x 6.5k..65k 333, now 119; 28 x 3.2k..32k 171, now 101; 16 x 8k (two items a head either way) 42, now 43.
constexpr int kDealSeqs = 256;
struct Deal {
  int items;      // all of them
  int wph;        // waves of an item
  ItemLoc it;     // this wave's item (n = 0: none)
  int seq, np[3]; // its sequence, that one's pages by type
};
// x / y of numbers below 2^20 (the compiler's integer division takes thirty instructions)
__device__ __forceinline__ int whole(int x, int y) { return uniform((int)(((float)x + 0.5f) * __builtin_amdgcn_rcpf((float)y))); }
template <int kFull>
__device__ inline Deal deal_item(const thinkv_view& v, const DecodeArgs& a, int wg, int wave) {
  constexpr int kU = kDealSeqs / 64;
  const thinkv_config& c = v.cfg;
  const int H = c.n_kv_heads, lane = threadIdx.x & 63;
  auto add = [](auto x, auto y) { return x + y; };
  int ids[kU], p[kU][3], tot[kU], most = 0;   // sequences lane, lane + 64, ..., their pages
  float all = 0.f;
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    ids[u] = 0;
    if (64 * u < a.B) ids[u] = a.seq_ids[min(64 * u + lane, a.B - 1)];
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    p[u][0] = p[u][1] = p[u][2] = 0;
    if (64 * u < a.B && 64 * u + lane < a.B && ids[u] >= 0 && ids[u] < c.max_seqs) {
#pragma unroll
      for (int k = 0; k < 3; ++k) p[u][k] = v.n_pages[npages_index(c, ids[u], a.layer, k)];
    }
  }
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    tot[u] = p[u][0] + p[u][1] + p[u][2];
    most = max(most, tot[u]);
    all += (float)tot[u];
  }
  most = last_lane(wave_scan(most, [](int x, int y) { return max(x, y); }));
  all = last_lane(wave_scan(all, add)) * (float)H;
  // (quotients by reciprocals: whatever n comes out of them, the sum decides whether it fits; what they are off by must not make
  // an item more of a whole number)
  const float per_most = __builtin_amdgcn_rcpf((float)max(most, 1)), per_all = __builtin_amdgcn_rcpf(fmaxf(all, 1.f));
  // the items of every sequence where the longest has n; their sum
  int mine[kU];
  auto spread = [&](int n) {
    const float per_page = (float)n * per_most;
    int sum = 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      mine[u] = 64 * u + lane < a.B ? min(max((int)ceilf(fmaf((float)tot[u], per_page, -0.002f)), 1), n) : 0;
      sum += mine[u];
    }
    return last_lane(wave_scan(sum, add));
  };
  int sub = 1, best_sub = kFull, best_n = 1, n = 0, sum = 0;
  float best = INFINITY;
  while (true) {
    const int slots = min(a.grid * sub, a.n_rows);
    if (slots >= a.B * H) {   // (holds for the last sub)
      const int least = kDealPages * whole(kFull, sub), cap = max(min(whole(min(most, 1 << 19) + least - 1, least), kMaxRowsPerHead), 1);
      n = max(min((int)(1.0001f * (float)slots * (float)most * per_all), cap), 1);
      for (sum = spread(n); n > 1 && sum * H > slots; sum = spread(n)) n = max(min(n - 1, whole(n * slots, sum * H)), 1);
      const float busiest = (float)most * (float)sub * __builtin_amdgcn_rcpf((float)n);
      if (busiest < 0.95f * best) {
        best = busiest;
        best_sub = sub;
        best_n = n;
      }
      // (n == cap: nothing to gain by smaller shares)
      if (best * (float)a.grid <= (sub == 1 && sum == n * a.B ? 1.3f : 1.08f) * all || n == cap) break;
    }
    if (sub == kFull) break;
    sub = kFull % (2 * sub) == 0 ? 2 * sub : kFull;
  }
  sub = uniform(best_sub);
  if (n != best_n) sum = spread(uniform(best_n));
  Deal d;
  d.items = sum * H;
  d.wph = whole(kFull, sub);
  d.it = ItemLoc{0, 0, 0, 0, 0};
  d.seq = -1;
  d.np[0] = d.np[1] = d.np[2] = 0;
  const int id = whole(wave, d.wph) * a.grid + wg;   // neighbouring items on different compute units
  if (id >= d.items) return d;
  int before = 0;
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    const int upto = before + wave_scan(mine[u], add), all_u = last_lane(upto);
    if (d.it.n == 0 && id < all_u * H) {
      const int at = __popcll(__ballot(upto * H <= id));   // (lanes without a sequence hold the same sum as the last one with)
      d.it.b = 64 * u + at;
      d.it.n = __builtin_amdgcn_readlane(mine[u], at);
      const int first = (__builtin_amdgcn_readlane(upto, at) - d.it.n) * H;
      d.it.j = whole(id - first, H);
      d.it.hkv = id - first - d.it.j * H;
      d.it.row0 = first + d.it.hkv * d.it.n;
#pragma unroll
      for (int k = 0; k < 3; ++k) d.np[k] = __builtin_amdgcn_readlane(p[u][k], at);
      d.seq = __builtin_amdgcn_readlane(ids[u], at);
    }
    before = all_u;
  }
  return d;
}

constexpr int kRowPad = 4;   // a partial row: acc[D], m, l, two unused words (rows stay 16-byte aligned)

__device__ inline float* partial_row(const DecodeArgs& a, int G, int D, int row, int g) {
  return a.partial + ((int64_t)row * G + g) * (D + kRowPad);
}

// Log-sum-exp merge of the partial rows of query head hq of query b, by D threads (first row and count as item 0 of the head left
// them); all threads of the workgroup come here together, those of no head (!on) with any head's number.
// Maxima and weights are found with one
// row per thread; the weighted sum over rows is unrolled so that several rows are in flight per thread.
template <int D>
struct MergeLds {
  float w[kMaxRowsPerHead];
  float red[D / 64];
};
template <int D>
__device__ __forceinline__ void merge_head(const thinkv_view& v, const DecodeArgs& a, int b, int hq, int ch, bool on, MergeLds<D>& lds) {
  const thinkv_config& c = v.cfg;
  const int Hq = c.n_q_heads, G = Hq / c.n_kv_heads, hkv = hq / G;
  const int row0 = a.alloc[2 * (b * c.n_kv_heads + hkv)];
  int ns = a.alloc[2 * (b * c.n_kv_heads + hkv) + 1];
  ns = ns > kMaxRowsPerHead ? kMaxRowsPerHead : ns;
  constexpr int RS = D + kRowPad;
  const float* src = partial_row(a, G, D, row0, hq % G);
  const int64_t stride = (int64_t)G * RS;   // from one row of this query head to the next
  // maximum over rows
  float m_loc = -INFINITY;
  for (int s = ch; s < ns; s += D) {
    const float m = src[s * stride + D];
    lds.w[s] = m;
    m_loc = fmaxf(m_loc, m);
  }
  for (int d = 32; d >= 1; d >>= 1) m_loc = fmaxf(m_loc, __shfl_xor(m_loc, d, 64));
  if ((ch & 63) == 0) lds.red[ch >> 6] = m_loc;
  __syncthreads();
  float M = lds.red[0];
  for (int w = 1; w < D / 64; ++w) M = fmaxf(M, lds.red[w]);
  __syncthreads();
  // weights and denominator
  float l_loc = 0.f;
  for (int s = ch; s < ns; s += D) {
    const float m = lds.w[s];
    const float f = (m == -INFINITY) ? 0.f : exp2f(m - M);
    lds.w[s] = f;
    l_loc = fmaf(src[s * stride + D + 1], f, l_loc);
  }
  for (int d = 32; d >= 1; d >>= 1) l_loc += __shfl_xor(l_loc, d, 64);
  if ((ch & 63) == 0) lds.red[ch >> 6] = l_loc;
  __syncthreads();
  float L = lds.red[0];
  for (int w = 1; w < D / 64; ++w) L += lds.red[w];
  // weighted sum of the partial rows
  float A = 0.f;
  const float* col = src + ch;
  int s = 0;
  for (; s + 4 <= ns; s += 4) {
    const float x0 = col[(s + 0) * stride], x1 = col[(s + 1) * stride];
    const float x2 = col[(s + 2) * stride], x3 = col[(s + 3) * stride];
    A = fmaf(x0, lds.w[s], A);
    A = fmaf(x1, lds.w[s + 1], A);
    A = fmaf(x2, lds.w[s + 2], A);
    A = fmaf(x3, lds.w[s + 3], A);
  }
  for (; s < ns; ++s) A = fmaf(col[s * stride], lds.w[s], A);
  if (!on) return;
  const float o = L > 0.f ? A / L : 0.f;
  store_from_f32(a.out, ((int64_t)b * Hq + hq) * D + ch, a.out_dtype, o);
  if (a.lse && ch == 0) a.lse[(int64_t)b * Hq + hq] = L > 0.f ? (M + log2f(L)) * 0.6931471805599453f : -INFINITY;
}

}  // namespace thinkv
