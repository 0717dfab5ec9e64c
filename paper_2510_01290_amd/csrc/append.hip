// Quantise-and-append: slot selection with in-place reuse of evicted slots, group
// quantisation of the new K/V rows, packing into the page layout, table updates.
//
// The result must equal a one-token-at-a-time loop (first reclaimable slot in list order,
// else the tail of the last page, else a new page popped in token order).  Because eviction
// never interleaves with an append call, that loop has a closed form per (sequence, type):
// the k-th token of the type (k counted inside the call) takes
//     k < R            the k-th reclaimable slot in (page, slot) order        (R = #reclaimable)
//     k < R + tail     slot filled + (k - R) of the last page                  (tail = 16 - filled)
//     otherwise        slot (k-R-tail) % 16 of the (k-R-tail)/16-th new page
// and new pages are granted to sequences in ascending sequence id, which is token order.
// Two kernels on the caller's stream:
//   plan   (block per sequence)  everything that concerns the sequence alone: token ranks per type, a place for every
//                                token, the masks, fill counts and the live count that follow from places in
//                                existing pages, and the new pages wanted
//   place  (block per token and share of its kv-heads, or per sixteen tokens)  quantisation, packing, slot_pos,
//                                handle.  Which page a new one is depends on the sequences before: it is worked out
//                                here, and the token that takes the page's first slot enters it into the tables.
// The place blocks use what the plan left in the workspace, the pools as the plan found them and the ids of pages that were there before,
// never an entry that the call writes, so nothing has to wait inside the kernel.  (settle asks for a page's id before it knows that the
// page was there: where it was not, another block may be writing the entry - one aligned word - and what was read is dropped.)  Small calls are bound by the two launches and chains of dependent loads, so
// the plan asks for everything that it can name at once and leaves a place ready for every token.  (With the tables left to
// the place kernel, which searched them for every token's slot, and to the last block of a sequence to arrive, or with
// a grant and a commit kernel behind more than 64 tokens: 16 tokens of 16 sequences of 32k, plan + place 20 us, now
// 14; 256 tokens of 256 sequences, a call, 34.6 us, now 17.2.)
// The grant of new pages (exclusive sum of the needs of the sequences before s, against what the
// pool held when the call began) is a sum over at most max_seqs small numbers: whoever wants it works it out for
// itself rather than waiting for a kernel of its own.  A decode step
// appends one token per sequence, so the call is a chain of short dependent launches and one
// launch less is a good part of its time.
#include "common.h"
#include "formats_dev.h"

#include <type_traits>

namespace thinkv {

struct SeqPlan {
  int lo, hi;        // token range of the sequence inside the call
  int n[3];          // tokens per type
  int old[3];        // reclaimable and never-used slots of the type's pages before the call: the first n tokens take them
  int np_old[3];
};
static_assert(sizeof(SeqPlan) == 11 * 4, "SeqPlan layout");

constexpr int kBulkFrom = 64;   // calls of more tokens take the bulk place kernel

// a token's place: state << 28 | index in the type's page list << 4 | slot
constexpr uint32_t kNoPlace = 0, kOldPage = 1, kNewPage = 2;
// In a bulk call one wave writes a new page whole if the call brings it at least so many tokens; fewer are stored by themselves, like
// those of existing pages (256 sequences, a new page each, us, by page and by token: one token 36 and 16, four 23.5 and 16.4, eight 19 and
// 17.8, twelve 20 and 19.8, sixteen 20.5 and 23.5).  A sequence that brings many tokens has three such pages at most: they are
// written whole too, rather than by a unit of sixteen rows in each block that holds some of their tokens (prompts of 1k to 4k tokens in
// the paper's formats 157 us, whole 150).
constexpr int kWholeFrom = 8, kManyTokens = 64;

struct AppendWs {
  SeqPlan* plan;     // [max_seqs]
  int* need;         // [3][max_seqs] new pages wanted (already limited by the page-list capacity)
  int* avail_old;    // [4]
  uint32_t* place;   // [n_tok]
};

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// What a caller is asked for is more than carve() takes: it has room for a count per page of every list, which an earlier
// layout kept, and callers hold workspaces of that size.
size_t append_ws_bytes(const thinkv_config& c, int n_tok) {
  return align256((size_t)c.max_seqs * 96) + 256 + align256((size_t)(n_tok > 0 ? n_tok : 1) * 4) +
         align256((size_t)c.max_seqs * 3 * c.max_pages * 4);
}

static AppendWs carve(const thinkv_config& c, int n_tok, void* ws) {
  static_assert(sizeof(SeqPlan) + 3 * sizeof(int) <= 96, "append_ws_bytes");
  char* p = (char*)ws;
  AppendWs w;
  w.plan = (SeqPlan*)p;
  w.need = (int*)(w.plan + c.max_seqs);
  p += align256((size_t)c.max_seqs * (sizeof(SeqPlan) + 3 * sizeof(int)));
  w.avail_old = (int*)p;
  p += 256;
  w.place = (uint32_t*)p;
  return w;
}

// three counts of at most 2^21 - 1 in one word
typedef unsigned long long Packed3;
__device__ __forceinline__ Packed3 pack3(int a, int b, int c) { return (Packed3)a | (Packed3)b << 21 | (Packed3)c << 42; }
__device__ __forceinline__ int part3(Packed3 x, int k) { return (int)(x >> (21 * k)) & 0x1FFFFF; }

template <int CTRL, int ROWS>
__device__ __forceinline__ Packed3 scan_step(Packed3 x) {
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWS, 0xF, false);
  return x + ((Packed3)hi << 32 | lo);
}

// inclusive scan over a wave: by 1, 2, 4, 8 lanes inside rows of sixteen, then the rows' sums onwards
__device__ __forceinline__ Packed3 wave_scan(Packed3 x) {
  x = scan_step<0x111, 0xF>(x);
  x = scan_step<0x112, 0xF>(x);
  x = scan_step<0x114, 0xF>(x);
  x = scan_step<0x118, 0xF>(x);
  x = scan_step<0x142, 0xA>(x);
  return scan_step<0x143, 0xC>(x);
}

// exclusive scans of N words per thread over a block of W waves, and the block's totals
template <int W, int N>
__device__ inline void block_excl_scan(const Packed3 (&v)[N], Packed3 (&excl)[N], Packed3 (&tot)[N], Packed3 (*lds)[W]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Packed3 inc[N];
#pragma unroll
  for (int i = 0; i < N; ++i) inc[i] = wave_scan(v[i]);
  __syncthreads();
  if (lane == 63)
#pragma unroll
    for (int i = 0; i < N; ++i) lds[i][wave] = inc[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    Packed3 off = 0;
    tot[i] = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const Packed3 t = lds[i][w];
      if (w < wave) off += t;
      tot[i] += t;
    }
    excl[i] = off + inc[i] - v[i];
  }
}

// Where the tokens of sequences below s end (bound 0) or those of sequences up to s (bound 1), by a wave: tok_seq does not
// decrease, so 256 probes at a time cut what is left into pieces, and the number of probes that lie before the bound
// says which piece has it.  (One thread halving the range takes fifteen dependent loads a bound for 35,000 tokens.)
__device__ inline int token_bound(const int32_t* __restrict__ tok_seq, int n_tok, int s, int bound) {
  int lo = 0, len = n_tok;   // the bound lies in [lo, lo + len]
  while (len > 0) {
    const int piece = (len + 255) / 256;
    int id[4], before = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) id[u] = tok_seq[lo + min((4 * (int)(threadIdx.x & 63) + u + 1) * piece, len) - 1];   // a piece's last element
#pragma unroll
    for (int u = 0; u < 4; ++u) before += __popcll(__ballot((4 * (int)(threadIdx.x & 63) + u) * piece < len && id[u] < s + bound));
    const int skip = min(before * piece, len);   // whole pieces before the bound
    lo += skip;
    len = skip >= len ? 0 : min(piece, len - skip) - 1;   // the next piece's last element does not lie before it
  }
  return lo;
}

constexpr int kKeep = 4;        // pages of a type a thread keeps the masks of (1,024 pages a list by 256 threads); longer lists are read again
constexpr int kWindow = 4096;   // tokens ranked at a time
// With more tokens than that per sequence slot of the view the plan takes 512 threads a sequence.  Fewer: the threads without a token only cost: 256 sequences, five
// tokens each, with their eviction, 19.9 us by 256 threads and 20.5 by 512.  The host does not know how many of the sequences bring tokens, so a prompt that comes
// alone into a view of many slots keeps 256: with the reset, 256 threads / 512, one of 300 tokens in 64 slots 22.2 / 18.3, of 8k 49.1 / 44.2, in 256 slots 50.3 / 45.3; but
// 64 prompts of 40 tokens in 256 slots 24.4 / 25.1, 4 of 64 in 64 18.0 / 18.7.
constexpr int kLongPrompts = 256;
constexpr int kEvAhead = 2;     // evictions of a call a thread holds before it applies the first
// (The plan is a chain of dependent loads: with handles, page counts, token ranges and last pages asked for one after the other behind
// the evictions it was eight long, now five.  256 sequences, a token out and a token in: plan 7.7 us, now 6.7, the call 15.7 and 14.5.)

__device__ __forceinline__ uint32_t page_mask(const uint32_t* msk, const uint32_t (&kept)[kKeep], int pi, int q0) {
  const int u = pi - q0;
  return u == 0 ? kept[0] : (u == 1 ? kept[1] : (u == 2 ? kept[2] : (u == 3 ? kept[3] : msk[pi])));
}

// T threads: 256, which have a token each up to that many and sixteen beyond, or 512, with one and eight.  (us a call, reset included, 256 / 512: 1 x 600 tokens
// 22.7 / 20.9, 1 x 8k 48.4 / 42.5, 16 x 1k..4k 80.0 / 77.4, 256 x 1k of 2 heads of 64 108 / 102; 1,024 have no registers for it: 33.9, 55.9, 89.7, 129.)
template <int T>
__global__ __launch_bounds__(T) void append_plan_kernel(thinkv_view v, int layer, const int32_t* __restrict__ tok_seq,
                                                          const uint8_t* __restrict__ tok_class, int n_tok, AppendWs ws,
                                                          const int32_t* __restrict__ ev_seq, const int32_t* __restrict__ ev_handle,
                                                          int n_ev) {
  __shared__ int s_rng[2];
  __shared__ Packed3 s_scan[4][T / 64];
  __shared__ uint16_t s_tok[kWindow];
  const thinkv_config& c = v.cfg;
  const int s = blockIdx.x, tid = threadIdx.x;
  // What does not depend on the evictions is asked for first: the page counts, the sequence's tokens (by two waves), the last
  // pages of the lists.
  int np_of[3], last_of[3], fill_of[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) np_of[k] = v.n_pages[npages_index(c, s, layer, k)];
  int ev_s[kEvAhead], ev_h[kEvAhead];
#pragma unroll
  for (int u = 0; u < kEvAhead; ++u) {
    const bool in = tid + T * u < n_ev;
    ev_s[u] = in ? ev_seq[tid + T * u] : s;
    ev_h[u] = in ? ev_handle[tid + T * u] : -1;
  }
  if (s == 0 && tid < 3) ws.avail_old[tid] = v.free_top[tid];   // the pools as the call finds them
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if (wave < 2) {
    if (n_tok <= kBulkFrom) {   // (a probe a token: one round)
      const uint64_t mine = __ballot(lane < n_tok && tok_seq[lane < n_tok ? lane : 0] == s);
      if (tid == 0) s_rng[0] = mine ? __builtin_ctzll(mine) : 0;
      if (tid == 64) s_rng[1] = mine ? 64 - __builtin_clzll(mine) : 0;
    } else {
      const int at = token_bound(tok_seq, n_tok, s, wave);
      if (lane == 0) s_rng[wave] = at;
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) last_of[k] = v.block_table[table_base(c, s, layer, k) + max(np_of[k] - 1, 0)];
  // Evictions that come with the call (thinkv_evict_append): an eviction touches the tables of its
  // own sequence only, and so does the plan of a sequence, so the block of sequence s applies the
  // handles of sequence s and goes on; no block waits for another.
  if (n_ev > 0) {
    auto evict = [&](int es, int32_t h) {
      if (es == s) evict_one(v, layer, s, h, np_of);
      else if (s == 0 && (es < 0 || es >= c.max_seqs)) atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
    };
#pragma unroll
    for (int u = 0; u < kEvAhead; ++u) evict(ev_s[u], ev_h[u]);
    for (int i = tid + T * kEvAhead; i < n_ev; i += T) evict(ev_seq[i], ev_handle[i]);
    __threadfence_block();
  }
  __syncthreads();
  const int lo = s_rng[0], hi = s_rng[1];
  SeqPlan pl;
  pl.lo = lo;
  pl.hi = hi;
#pragma unroll
  for (int k = 0; k < 3; ++k) pl.n[k] = pl.old[k] = pl.np_old[k] = 0;
  if (lo >= hi) {
    if (tid == 0) ws.plan[s] = pl;
    if (tid < 3) ws.need[tid * c.max_seqs + s] = 0;
    return;
  }
  // ---- reclaimable slots: every thread takes a contiguous run of pages of every type.  (Loads without branches around them:
  // all are under way at once, with those of the last pages' fill counts and of the tokens' types.)
  int q0[3], q1[3], first[3], have[3], R[3];
  uint32_t kept[3][kKeep];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int64_t row = table_base(c, s, layer, k);
    const int np = np_of[k], per = (np + T - 1) / T;
    q0[k] = min(tid * per, np);
    q1[k] = min(q0[k] + per, np);
#pragma unroll
    for (int u = 0; u < kKeep; ++u) kept[k][u] = v.slot_mask[row + min(q0[k] + u, c.max_pages - 1)];
  }
  // ---- tokens, a window at a time: every token's rank among the call's tokens of its type.  A token behind the reclaimable
  // slots knows its place from its rank; the others are listed by rank and get it from the thread that has the slot's page.
  int n[3] = {0, 0, 0};
  auto window = [&](auto per_thread, int w0) {
    constexpr int U = decltype(per_thread)::value;
    const int t0 = w0 + tid * U;
    int cl[U], mine[3] = {0, 0, 0}, rank[3], cnt[3];
#pragma unroll
    for (int u = 0; u < U; ++u) cl[u] = (int)tok_class[min(t0 + u, hi - 1)];
    if (w0 == lo) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        fill_of[k] = np_of[k] > 0 ? (int)v.page_filled[k][last_of[k]] : kPage;
        have[k] = 0;
#pragma unroll
        for (int u = 0; u < kKeep; ++u) {
          kept[k][u] = q0[k] + u < q1[k] ? kept[k][u] : 0u;
          have[k] += __popc(kept[k][u] >> 16);
        }
        for (int pi = q0[k] + kKeep; pi < q1[k]; ++pi) have[k] += __popc(v.slot_mask[table_base(c, s, layer, k) + pi] >> 16);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      cl[u] = t0 + u < hi ? cl[u] : 3;
#pragma unroll
      for (int k = 0; k < 3; ++k) mine[k] += cl[u] == k;
    }
    // the window's tokens of each type together, the reclaimable slots apart (there may be more than a packed word holds)
    const Packed3 x[4] = {pack3(mine[0], mine[1], mine[2]), (Packed3)have[0], (Packed3)have[1], (Packed3)have[2]};
    Packed3 ex[4], tot[4];
    block_excl_scan<T / 64>(x, ex, tot, s_scan);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      rank[k] = part3(ex[0], k);
      cnt[k] = part3(tot[0], k);
      first[k] = (int)ex[k + 1];
      R[k] = (int)tot[k + 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint32_t at = kNoPlace << 28;
      bool listed = false;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (cl[u] != k) continue;
        const int r = n[k] + rank[k], kk = r - R[k] - (kPage - fill_of[k]);
        if (r < R[k]) {
          s_tok[(k > 0 ? cnt[0] : 0) + (k > 1 ? cnt[1] : 0) + rank[k]] = (uint16_t)(tid * U + u);
          listed = true;
        } else if (kk < 0) {
          at = kOldPage << 28 | (uint32_t)(np_of[k] - 1) << 4 | (uint32_t)(kk + kPage);
        } else {
          const int pi = np_of[k] + (kk >> 4);   // never granted beyond the page list
          at = kNewPage << 28 | (uint32_t)(pi < c.max_pages ? pi : c.max_pages) << 4 | (uint32_t)(kk & 15);
        }
        ++rank[k];
      }
      if (t0 + u < hi && !listed) ws.place[t0 + u] = at;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int off = (k > 0 ? cnt[0] : 0) + (k > 1 ? cnt[1] : 0) - n[k];
      const int r0 = max(first[k], n[k]), r1 = min(first[k] + have[k], n[k] + cnt[k]);   // the window's ranks on this thread's pages
      int r = first[k];
      for (int pi = q0[k]; r0 < r1 && pi < q1[k] && r < r1; ++pi) {
        uint32_t e = page_mask(v.slot_mask + table_base(c, s, layer, k), kept[k], pi, q0[k]) >> 16;
        for (; e && r < r1; e &= e - 1, ++r)
          if (r >= r0) ws.place[w0 + s_tok[off + r]] = kOldPage << 28 | (uint32_t)pi << 4 | (uint32_t)(__ffs(e) - 1);
      }
    }
    __syncthreads();   // (the list is rewritten)
#pragma unroll
    for (int k = 0; k < 3; ++k) n[k] += cnt[k];
  };
  if (hi - lo <= T) window(std::integral_constant<int, 1>(), lo);
  else
    for (int w0 = lo; w0 < hi; w0 += kWindow) window(std::integral_constant<int, kWindow / T>(), w0);
  // ---- what follows for the pages the sequence has: the first n of the reclaimable, then of the never-used slots are live
  int placed = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int np = np_of[k], fill = fill_of[k], old = R[k] + kPage - fill;
    int need = n[k] > old ? (n[k] - old + kPage - 1) / kPage : 0;
    need = min(need, c.max_pages - np);
    pl.n[k] = n[k];
    pl.old[k] = old;
    pl.np_old[k] = np;
    if (tid == 0) ws.need[k * c.max_seqs + s] = need;
    placed += min(n[k], old);
    uint32_t* const msk = v.slot_mask + table_base(c, s, layer, k);
    const int add = n[k] > R[k] ? min(n[k] - R[k], kPage - fill) : 0;   // never-used slots of the last page that are taken
    int left = n[k] - first[k];   // slots to take from this thread's pages
    for (int pi = q0[k]; pi < q1[k]; ++pi) {
      const bool tail = add > 0 && pi == np - 1;
      if (left <= 0 && add == 0) break;
      uint32_t m = page_mask(msk, kept[k], pi, q0[k]);
      const uint32_t before = m;
      for (uint32_t e = m >> 16; e && left > 0; e &= e - 1, --left) {
        const uint32_t bit = e & (0u - e);
        m = (m | bit) & ~(bit << 16);
      }
      if (tail) {
        m |= ((1u << add) - 1u) << fill;
        v.page_filled[k][last_of[k]] = (uint8_t)(fill + add);
      }
      if (m != before) msk[pi] = m;
    }
  }
  if (tid == 0) {
    ws.plan[s] = pl;
    if (placed) v.n_live[sl_index(c, s, layer)] += placed;
  }
}

// New pages of type k granted to sequence s: base = pages wanted by the sequences before s (pop order), grant = what the pool
// (avail pages when the call began) still covers of s's own need.  Called by LPT neighbouring lanes together.
template <int LPT>
__device__ inline void grant_of(const AppendWs& ws, int n_seqs, int s, int k, int* base, int* grant) {
  const int avail = ws.avail_old[k];
  const int* const need = ws.need + k * n_seqs;
  int before = 0;
  for (int t = threadIdx.x & (LPT - 1); t < s; t += 8 * LPT) {   // eight loads at once
    int x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = need[min(t + u * LPT, s)];
#pragma unroll
    for (int u = 0; u < 8; ++u) before += t + u * LPT < s ? x[u] : 0;
  }
#pragma unroll
  for (int d = LPT / 2; d >= 1; d >>= 1) before += __shfl_xor(before, d, 64);
  const int left = avail - before;
  *base = before < avail ? before : avail;
  *grant = left < 0 ? 0 : (left < need[s] ? left : need[s]);
}

// One token's place, by LPT neighbouring lanes: type, page, slot, page list index; ok = 0 if it gets none; cnt = tokens that the
// call puts into the page, if it is a new one.  enter: these lanes also record it (slot_pos, handle) and, for a token in a new
// page, enter the page into the tables: the token in the page's first slot writes the page's row, the first token of
// the type that wants a new page the counts.  BULK: the positions of the tokens of a page that is written whole are left to who writes it.
struct Place {
  int ok, cls, pid, slot, pi, cnt, whole;   // whole: the page is written as one
};
template <int LPT, bool BULK>
__device__ inline Place settle(const thinkv_view& v, int layer, const AppendWs& ws, const int32_t* __restrict__ tok_seq, const int32_t* __restrict__ tok_pos,
                               const uint8_t* __restrict__ tok_class, int32_t* __restrict__ tok_handle, int i, bool enter) {
  const thinkv_config& c = v.cfg;
  const int lane = threadIdx.x & (LPT - 1);
  const int s = tok_seq[i];
  const int cls = tok_class[i];
  const uint32_t at = ws.place[i];
  const int pos = tok_pos[i];
  Place p = {0, cls > 2 ? 0 : cls, 0, 0, 0, 0, 0};
  if (s < 0 || s >= c.max_seqs) {
    if (enter && lane == 0) atomicOr(&v.dev_status[c.max_seqs * c.n_layers], THINKV_ST_BAD_SEQ);
  } else {
    const SeqPlan& pl = ws.plan[s];
    // (The page's id is asked for beside the plan that says whether it is the token's; a new page's entry may be under way meanwhile, and is
    // not used.  Relaxed atomics on both sides, or asking only where the place says that the page was there, cost 256 sequences
    // 14.5 to 14.8 us a call instead of 14.35.)
    const int listed = (int)(at >> 4) & 0xFFFFFF;
    const int old_pid = v.block_table[table_base(c, s, layer, p.cls) + (listed < c.max_pages ? listed : 0)];
    if (cls > 2) {
      if (enter && lane == 0) atomicOr(&v.dev_status[sl_index(c, s, layer)], THINKV_ST_BAD_CLASS);
    } else if (i >= pl.lo && i < pl.hi) {   // (outside: the sequence ids of the call decrease somewhere)
      const uint32_t state = at >> 28;
      p.slot = at & 15;
      p.pi = (at >> 4) & 0xFFFFFF;
      const int npi = p.pi - pl.np_old[cls];
      if (state == kOldPage && npi < 0) {
        p.ok = 1;
        p.pid = old_pid;
      } else if (state == kNewPage && npi >= 0) {
        int base, grant;
        grant_of<LPT>(ws, c.max_seqs, s, cls, &base, &grant);
        const int n_new = pl.n[cls] - pl.old[cls];
        if (npi < grant) {
          p.ok = 1;
          p.pid = v.free_stack[cls][ws.avail_old[cls] - 1 - (base + npi)];
        }
        p.cnt = n_new - kPage * npi < kPage ? n_new - kPage * npi : kPage;
        p.whole = BULK && (p.cnt >= kWholeFrom || pl.hi - pl.lo >= kManyTokens);
        if (enter && p.slot == 0) {
          if (p.ok) {
            if (lane == 0) {
              const int64_t row = table_base(c, s, layer, cls) + p.pi;
              v.block_table[row] = p.pid;
              v.slot_mask[row] = (1u << p.cnt) - 1u;
              v.page_filled[cls][p.pid] = (uint8_t)p.cnt;
            }
            if (!p.whole)
              for (int sl = p.cnt + lane; sl < kPage; sl += LPT) v.slot_pos[cls][(int64_t)p.pid * kPage + sl] = -1;
          }
          if (npi == 0 && lane == 0) {
            if (grant > 0) {
              v.n_pages[npages_index(c, s, layer, cls)] = pl.np_old[cls] + grant;
              atomicAdd(&v.n_live[sl_index(c, s, layer)], n_new < kPage * grant ? n_new : kPage * grant);
            }
            if (n_new > kPage * grant) atomicOr(&v.dev_status[sl_index(c, s, layer)], THINKV_ST_NOPAGES);
          }
        }
      }
    }
  }
  if (enter && lane == 0) {
    if (p.ok && !p.whole) {
      v.slot_pos[p.cls][(int64_t)p.pid * kPage + p.slot] = pos;
      atomicMax(&v.page_pos_max[p.cls][p.pid], pos);
    }
    if (tok_handle) tok_handle[i] = p.ok ? THINKV_HANDLE(p.cls, p.pi, p.slot) : -1;
  }
  return p;
}

// The pools after the call: what all sequences together were granted is gone.  (One wave; nothing in the call reads free_top
// after the plan kernel's snapshot.)
__device__ inline void update_pools(const thinkv_view& v, const AppendWs& ws) {
  const int lane = threadIdx.x & 63;
  for (int k = 0; k < 3; ++k) {
    int want = 0;
    for (int t = lane; t < v.cfg.max_seqs; t += 512) {
      int x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = ws.need[k * v.cfg.max_seqs + min(t + 64 * u, v.cfg.max_seqs - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) want += t + 64 * u < v.cfg.max_seqs ? x[u] : 0;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) want += __shfl_xor(want, d, 64);
    const int avail = ws.avail_old[k];
    if (lane == 0) v.free_top[k] = avail - (want < avail ? want : avail);
  }
}

// Codes of a group in the integer formats: code = clamp(rint((x - zp) / s), 0, qmax) with IEEE's quotient, s = (max - min) / qmax
// rounded up to binary16.  Both divisors have few significant bits, eleven and at most eight: the quotient of a binary32 number by such
// a number is never within 2^-12 of a unit in the last place of the middle between two neighbouring numbers, so a
// reciprocal good to a unit in the last place, one product and one residual correction (exact: its terms have a dozen bits
// in common) give the correctly rounded quotient: three instructions in place of the eleven of a division (37,000 tokens of 16 prompts,
// with the reset, 93 us with divisions and 81 so; 256 tokens of 256 sequences 16.1 and 15.6).  That
// needs finite numbers.  Otherwise the division's result is one of two for the whole group, and numbers in place of zp,
// s and 1 / s make the same three instructions give it: code 0 if the scale is 0 or not finite (or the zero-point is not a number or
// +inf), and the highest code if the zero-point is -inf.  A value that is not a number gets code 0.
struct GroupCode {
  float sf, zf, r;
  uint32_t meta;   // scale | zero-point << 16
};
__device__ __forceinline__ GroupCode group_code(float mn, float mx, float qmax, float inv_qmax) {
  const _Float16 zp = (_Float16)(mn + 0.0f);
  const float range = mx - mn, s0 = range * inv_qmax;
  const float s32 = range < INFINITY ? fmaf(fmaf(-qmax, s0, range), inv_qmax, s0) : range;
  const _Float16 near = (_Float16)s32;
  const uint16_t sc = (uint16_t)(__builtin_bit_cast(uint16_t, near) + ((float)near < s32 ? 1 : 0));
  GroupCode g;
  g.sf = (float)__builtin_bit_cast(_Float16, sc);
  g.zf = (float)zp;
  g.r = __builtin_amdgcn_rcpf(g.sf);
  g.meta = (uint32_t)sc | (uint32_t)__builtin_bit_cast(uint16_t, zp) << 16;
  const bool scale = g.sf > 0.0f && g.sf < INFINITY;
  if (!(scale && fabsf(g.zf) < INFINITY)) {
    const bool top = scale && g.zf == -INFINITY;
    g.zf = top ? g.zf : 0.0f;
    g.sf = top ? -1.0f : 0.0f;
    g.r = top ? 1.0f : 0.0f;
  }
  return g;
}
// (The middle of three with a NaN is the smaller of the other two.  With a finite scale differences stay below 2^25, but for an
// infinity whose group's maximum a signalling NaN has swallowed: the first clamp keeps it out of the correction.)  The result is what the
// conversion to a byte rounds (v_cvt_pk_u8_f32: to nearest, ties to even).
__device__ __forceinline__ float group_quotient(const GroupCode& g, float x, float qmax) {
  const float d = __builtin_amdgcn_fmed3f(x - g.zf, -0x1p60f, 0x1p60f);
  const float q0 = d * g.r;
  const float q = fmaf(fmaf(-g.sf, q0, d), g.r, q0);
  return __builtin_amdgcn_fmed3f(q, 0.0f, qmax);
}
// 1 / (2^bits - 1), as a division gives it
__device__ __forceinline__ float inverse_of_qmax(int bits) { return bits == 2 ? 1.0f / 3.0f : (bits == 4 ? 1.0f / 15.0f : 1.0f / 255.0f); }

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E;   // lane ^ 1 and lane ^ 2 of a quad

// A row piece: eight channels of a group of 32, whose four pieces are held by four neighbouring lanes.  Returns the codes, one a
// byte.
__device__ __forceinline__ uint2 piece_codes(const float (&x)[8], float qmax, float inv_qmax, uint32_t* meta) {
  float mn = x[0], mx = x[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) {
    mn = fminf(mn, x[e]);
    mx = fmaxf(mx, x[e]);
  }
  mn = fminf(mn, dpp<kDppXor1>(mn));
  mx = fmaxf(mx, dpp<kDppXor1>(mx));
  mn = fminf(mn, dpp<kDppXor2>(mn));
  mx = fmaxf(mx, dpp<kDppXor2>(mx));
  const GroupCode g = group_code(mn, mx, qmax, inv_qmax);
  *meta = g.meta;
  uint2 w = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    w.x = __builtin_amdgcn_cvt_pk_u8_f32(group_quotient(g, x[e], qmax), e, w.x);
    w.y = __builtin_amdgcn_cvt_pk_u8_f32(group_quotient(g, x[4 + e], qmax), e, w.y);
  }
  return w;
}

// The same in the paper's formats: the eight channels lie in one group of 16, which two neighbouring lanes share; ratios to the
// scale in binary64, as the formats are defined.  whole_scale: the tensor-wide scale of the 8-bit format.
__device__ __forceinline__ uint2 piece_codes_fp(const float (&x)[8], int bits, double whole_scale, uint32_t* meta) {
  double sd = whole_scale;
  if (bits != 8) {
    float amax = fabsf(x[0]);
#pragma unroll
    for (int e = 1; e < 8; ++e) amax = fmaxf(amax, fabsf(x[e]));
    amax = fmaxf(amax, dpp<kDppXor1>(amax));
    *meta = e4m3_code_up((double)amax / (bits == 4 ? 6.0 : 1.0));
    sd = (double)e4m3_value(*meta);
  }
  uint32_t code[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const double r = sd > 0.0 ? (double)x[e] / sd : 0.0;
    code[e] = bits == 8 ? e4m3_encode(r) : (bits == 4 ? e2m1_encode(r) : ternary_encode(r));
  }
  uint2 w = {0u, 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    w.x |= code[e] << (8 * e);
    w.y |= code[4 + e] << (8 * e);
  }
  return w;
}

// K codes of piece j of group grp: channel 32 grp + 8 j + e is field 4 grp + e / 2, half e % 2, of the chunk.
__device__ __forceinline__ void put_k(uint8_t* chunk, int bits, int grp, uint2 w) {
  if (bits == 8) {          // fields 4 grp .. + 3 are words 2 grp and 2 grp + 1
    *(uint2*)(chunk + 8 * grp) = uint2{__builtin_amdgcn_perm(0u, w.x, 0x03010200u), __builtin_amdgcn_perm(0u, w.y, 0x03010200u)};
    return;
  }
  const uint32_t even = __builtin_amdgcn_perm(w.y, w.x, 0x05010400u), odd = __builtin_amdgcn_perm(w.y, w.x, 0x07030602u);   // codes 0 4 1 5, 2 6 3 7
  if (bits == 4) {          // word grp
    *(uint32_t*)(chunk + 4 * grp) = even | odd << 4;
  } else {                  // a quarter of each half of word grp / 2
    const uint32_t two = even | odd << 2, four = two | two >> 4;
    chunk[4 * (grp >> 1) + (grp & 1)] = (uint8_t)four;
    chunk[4 * (grp >> 1) + 2 + (grp & 1)] = (uint8_t)(four >> 16);
  }
}

// ---------------------------------------------------------------------------------------------
// place: one block per (token, share of the kv-heads); every block of a token derives the same
// place, block 0 records it.
template <int D>
__global__ __launch_bounds__(256) void append_place_kernel(thinkv_view v, int layer, const void* __restrict__ k_new,
                                                           const void* __restrict__ v_new, const int32_t* __restrict__ tok_seq,
                                                           const int32_t* __restrict__ tok_pos, const uint8_t* __restrict__ tok_class,
                                                           int32_t* __restrict__ tok_handle, int n_tok, int in_dtype, AppendWs ws,
                                                           int heads_per_block) {
  constexpr int NG = D / kGroup;        // groups per row
  constexpr int NM = D / 16;            // 16-channel blocks per row
  constexpr int HP = 256 / (2 * D);     // heads handled per pass
  __shared__ int s_place[4];            // type, page id, slot, ok
  __shared__ uint8_t s_codes[HP][2][D];
  __shared__ uint32_t s_meta[HP][2][NG];
  __shared__ uint8_t s_scale8[HP][2][D / kGroupFp];   // THINKV_FMT_FP: the E4M3 scale codes of the row's groups of 16
  const thinkv_config& c = v.cfg;
  const int i = blockIdx.x, tid = threadIdx.x;
  // the first input value of this thread is requested before the slot is settled: the slot takes a
  // chain of dependent loads, and a decode-style call is nothing but latency
  const int hs = tid / (2 * D), r = tid % (2 * D), kind = r / D, ch = r % D;
  const int h_first = blockIdx.y * heads_per_block + hs;
  const int h_end = (int)(blockIdx.y + 1) * heads_per_block < c.n_kv_heads ? (int)(blockIdx.y + 1) * heads_per_block : c.n_kv_heads;
  float x_first = 0.f;
  if (h_first < h_end) x_first = load_as_f32(kind ? v_new : k_new, ((int64_t)i * c.n_kv_heads + h_first) * D + ch, in_dtype);
  if (tid < 64) {
    const Place p = settle<64, false>(v, layer, ws, tok_seq, tok_pos, tok_class, tok_handle, i, blockIdx.y == 0);
    if (tid == 0) {
      s_place[0] = p.cls; s_place[1] = p.pid; s_place[2] = p.slot; s_place[3] = p.ok;
    }
  } else if (tid < 128 && blockIdx.x == 0 && blockIdx.y == 0) {
    update_pools(v, ws);
  }
  __syncthreads();
  if (!s_place[3]) return;
  const int cls = s_place[0], pid = s_place[1], t = s_place[2];
  const int bits = c.bits_of_class[cls];
  const bool fp = c.format == THINKV_FMT_FP;
  const BlockGeom g = block_geom(bits, D, c.format);
  const int H = c.n_kv_heads;
  const float qmax = (float)((1 << bits) - 1);
  uint8_t* page = v.arena[cls] + (int64_t)pid * H * g.block_bytes;
  // (all powers of two: quotients are shifts)
  const int lb = bits == 2 ? 1 : (bits == 4 ? 2 : 3), lc = lb + (D == 128 ? 2 : 1);   // logarithms of the width and of a chunk's bytes
  const int CB = 1 << lc, CPB = 8 >> lb;  // bytes of a chunk, codes per byte

  for (int h0 = blockIdx.y * heads_per_block; h0 < h_end; h0 += HP) {
    const int h = h0 + hs;
    if (h < h_end) {
      const void* src = kind ? v_new : k_new;
      const float x = h == h_first ? x_first : load_as_f32(src, ((int64_t)i * H + h) * D + ch, in_dtype);
      if (fp) {
        // the paper's formats: the ratio to the scale in binary64, as the formats are defined
        uint32_t code;
        if (bits == 8) {
          code = e4m3_encode((double)x / (double)c.fp8_scale[kind]);
        } else {
          float amax = fabsf(x);
#pragma unroll
          for (int d = 8; d >= 1; d >>= 1) amax = fmaxf(amax, __shfl_xor(amax, d, 64));
          const uint32_t sc8 = e4m3_code_up((double)amax / (bits == 4 ? 6.0 : 1.0));
          const double sd = (double)e4m3_value(sc8);
          const double r = sd > 0.0 ? (double)x / sd : 0.0;
          code = bits == 4 ? e2m1_encode(r) : ternary_encode(r);
          if ((ch & 15) == 0) s_scale8[hs][kind][ch >> 4] = (uint8_t)sc8;
        }
        s_codes[hs][kind][ch] = (uint8_t)code;
      } else {
      float mn = x, mx = x;
#pragma unroll
      for (int d = 16; d >= 1; d >>= 1) {
        mn = fminf(mn, __shfl_xor(mn, d, 64));
        mx = fmaxf(mx, __shfl_xor(mx, d, 64));
      }
      const GroupCode gc = group_code(mn, mx, qmax, inverse_of_qmax(bits));
      s_codes[hs][kind][ch] = (uint8_t)__builtin_amdgcn_cvt_pk_u8_f32(group_quotient(gc, x, qmax), 0, 0u);
      if ((ch & 31) == 0)
        s_meta[hs][kind][ch >> 5] = gc.meta;
      }
    }
    __syncthreads();
    // pack: every destination byte the slot owns is assembled by one thread
    const int per_head = 8 * CB;  // 4*CB bytes of K codes + 4*CB bytes of V codes
    const int ph = tid >> (lc + 3), pr = tid & (per_head - 1);
    if (ph < HP && h0 + ph < H) {
      uint8_t* blk = page + (int64_t)(h0 + ph) * g.block_bytes;
      uint32_t byte = 0;
      if (pr < 4 * CB) {  // K: chunk 16*j + t, byte ob
        const int j = pr >> lc, ob = pr & (CB - 1);
        const int w = ob >> 2, bo = (ob & 3) * 8, hh = bo >> 4, lf = (bo & 15) >> lb;
        for (int q = 0; q < CPB; ++q) {
          const int f = (w << (4 - lb)) + lf + q;
          const int chn = 32 * (f >> 2) + 8 * j + 2 * (f & 3) + hh;
          byte |= (uint32_t)s_codes[ph][0][chn] << (q * bits);
        }
        blk[g.k_codes + (16 * j + t) * CB + ob] = (uint8_t)byte;
      } else {            // V: chunk 16*(t/4) + m, fields u*NM .. u*NM+NM-1 of half t%2
        const int vb = pr - 4 * CB, lo = lc - 2;   // CB / 4 bytes of a slot in a chunk
        const int m = vb >> lo, kk = vb & ((1 << lo) - 1);
        const int u = (t >> 1) & 1, hh = t & 1;
        const int f0 = u * NM + kk * CPB;
        const int off = 4 * (f0 >> (4 - lb)) + 2 * hh + (((f0 & ((16 >> lb) - 1)) << lb) >> 3);
        for (int q = 0; q < CPB; ++q) {
          const int mb = kk * CPB + q;
          byte |= (uint32_t)s_codes[ph][1][16 * mb + m] << (q * bits);
        }
        blk[g.v_codes + (16 * (t >> 2) + m) * CB + off] = (uint8_t)byte;
      }
    }
    if (fp) {
      constexpr int NG16 = D / kGroupFp;
      if (bits != 8 && tid < HP * 2 * NG16) {
        const int mh = tid / (2 * NG16), mr = tid % (2 * NG16), mk = mr / NG16, mg = mr % NG16;
        if (h0 + mh < H) (page + (int64_t)(h0 + mh) * g.block_bytes)[(mk ? g.v_meta : g.k_meta) + mg * kPage + t] = s_scale8[mh][mk][mg];
      }
    } else if (tid < HP * 2 * NG) {
      const int mh = tid / (2 * NG), mr = tid % (2 * NG), mk = mr / NG, mg = mr % NG;
      if (h0 + mh < H) {
        uint8_t* blk = page + (int64_t)(h0 + mh) * g.block_bytes;
        const uint32_t md = s_meta[mh][mk][mg];
        uint16_t* meta = (uint16_t*)(blk + (mk ? g.v_meta : g.k_meta));
        meta[meta_index(t, mg)] = (uint16_t)(md & 0xFFFFu);
        meta[meta_index(t, mg) + 4] = (uint16_t)(md >> 16);
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Bulk calls (prefill-style: thousands of tokens).  A block takes sixteen consecutive tokens of the call and settles their
// places side by side, sixteen lanes a token.  The unit of work behind that is the K or the V rows of sixteen tokens and one
// kv-head, by one wave: eight channels a lane (one 16-byte load), codes in registers, V codes transposed through LDS (a V
// chunk holds channels 16 apart).
// New pages are written whole: the token in a new page's first slot brings the page to its block, the others are the next
// fifteen of its type, and the unit's part of the page (0.3 to 2.3 KB) is put together in LDS and stored in 16-byte words.
// Tokens that take slots of existing pages are stored field by field.
// What bounds it: reading the rows, 256 bytes at a time, and next to that the vector instructions of the quantiser (with
// divisions in it the kernel is a fifth longer).  Leaving things out of its 58 us: the rows' loads 45, the pages' stores 54, the quantiser 47, all of
// these 28, and everything but the places 15.
// 37,000 tokens of 16 prompts, 8 kv-heads of 128, bf16 (151 MB in, 50 MB out): 96.5 us with a block of sixteen tokens
// storing 2 to 8 bytes at a time into pages that four blocks shared, 67 with whole pages, 60 with nontemporal loads of
// neighbouring heads side by side.  Rows requested a unit ahead gained nothing (64 against 60), nor did K and V in one unit (more
// registers, fewer waves).
constexpr int kBulkTokens = 16;   // tokens per block of the bulk place kernel

// A new page: its first token in the call, type, number, tokens the call puts into it, the end of the sequence's tokens.
struct NewPage {
  int first, cls, pid, cnt, end;
};

// LDS of a wave: the K or V part of a block (codes, scales), and the V codes of sixteen rows, one a byte
template <int D>
struct UnitLds {
  uint4 codes[(D == 128 ? 2048 : 1024) / 16];
  uint4 meta[(D == 128 ? 256 : 128) / 16];
  uint32_t v[kPage][D / 4];
};

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int IN>
__device__ __forceinline__ void widen(const uint4* raw, float (&x)[8]) {
  const uint4 r0 = raw[0], r1 = raw[IN == THINKV_F32 ? 1 : 0];
  const uint32_t w[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
  if (IN == THINKV_F32) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __builtin_bit_cast(float, w[e]);
  } else if (IN == THINKV_F16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w[e >> 1] >> (16 * (e & 1))));
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __builtin_bit_cast(float, e & 1 ? w[e >> 1] & 0xFFFF0000u : w[e >> 1] << 16);
  }
}

// Sixteen bytes that are read once (nontemporal: they leave the caches to the pages).
__device__ __forceinline__ uint4 load_once(const void* p) {
  typedef uint32_t Word4 __attribute__((ext_vector_type(4)));
  const Word4 w = __builtin_nontemporal_load((const Word4*)p);
  return uint4{w.x, w.y, w.z, w.w};
}

// What a row of a unit is: its token, and the page and slot it goes to.
struct Row {
  int tok, cls, pid, slot;
};

// The K (kind 0) or V (kind 1) rows of sixteen tokens and kv-head h, by a wave.  WHOLE: the rows are the slots of one new page, of
// which the first cnt are taken.  Otherwise row r goes to its own page if bit r of rows is set.
template <int D, int IN, bool FP, bool WHOLE, typename RowOf>
__device__ __forceinline__ void place_unit(const thinkv_view& v, const void* __restrict__ src, int kind, int h, RowOf row_of, uint32_t rows, UnitLds<D>& lds) {
  constexpr int NM = D / 16, TPR = D / 8, RP = 64 / TPR, NP = kPage / RP, kW = IN == THINKV_F32 ? 2 : 1;
  const thinkv_config& c = v.cfg;
  const int lane = threadIdx.x & 63, H = c.n_kv_heads;
  const int piece = lane % TPR, grp = piece >> 2, j = piece & 3;
  uint4 raw[NP][kW];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = RP * p + lane / TPR;
    const int i = row_of(rows >> r & 1 ? r : __builtin_ctz(rows)).tok;   // (rows that are not there are quantised and not stored)
    const int64_t at = ((int64_t)i * H + h) * D + 8 * piece;
#pragma unroll
    for (int w = 0; w < kW; ++w)
      raw[p][w] = load_once(IN == THINKV_F32 ? (const void*)((const float*)src + at + 4 * w) : (const void*)((const uint16_t*)src + at));
  }
  // WHOLE: the page's two parts
  uint4 *page_codes = nullptr, *page_meta = nullptr;
  int n_codes = 0, n_meta = 0;
  if (WHOLE) {
    const Row row = row_of(0);
    const BlockGeom g = block_geom(c.bits_of_class[row.cls], D, c.format);
    uint8_t* const blk = v.arena[row.cls] + ((int64_t)row.pid * H + h) * g.block_bytes;
    page_codes = (uint4*)(blk + (kind ? g.v_codes : g.k_codes));
    page_meta = (uint4*)(blk + (kind ? g.v_meta : g.k_meta));
    n_codes = 4 * g.chunk_bytes;                                    // 64 chunks
    n_meta = (g.block_bytes - 2 * 64 * g.chunk_bytes) / 2 / 16;
    if (rows != 0xFFFFu) {   // a page that stays partly empty keeps what its other slots hold
      for (int w = lane; w < n_codes; w += 64) lds.codes[w] = page_codes[w];
      for (int w = lane; w < n_meta; w += 64) lds.meta[w] = page_meta[w];
    }
    wave_lds_order();
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = RP * p + lane / TPR;
    const Row row = row_of(r);
    const int bits = c.bits_of_class[row.cls];
    const float qmax = (float)((1 << bits) - 1);
    float x[8];
    widen<IN>(raw[p], x);
    uint32_t meta = 0;
    const uint2 w = FP ? piece_codes_fp(x, bits, (double)c.fp8_scale[kind], &meta) : piece_codes(x, qmax, inverse_of_qmax(bits), &meta);
    if (rows >> r & 1) {
      const BlockGeom g = block_geom(bits, D, c.format);
      uint8_t* const blk = WHOLE ? nullptr : v.arena[row.cls] + ((int64_t)row.pid * H + h) * g.block_bytes;
      if (!kind) put_k((WHOLE ? (uint8_t*)lds.codes : blk + g.k_codes) + (16 * j + row.slot) * g.chunk_bytes, bits, grp, w);
      else *(uint2*)&lds.v[r][2 * piece] = w;
      uint8_t* const m = WHOLE ? (uint8_t*)lds.meta : blk + (kind ? g.v_meta : g.k_meta);
      if (FP) {
        if (bits != 8 && (j & 1) == 0) m[(2 * grp + (j >> 1)) * kPage + row.slot] = (uint8_t)meta;
      } else if (j == 0) {
        ((uint16_t*)m)[meta_index(row.slot, grp)] = (uint16_t)meta;
        ((uint16_t*)m)[meta_index(row.slot, grp) + 4] = (uint16_t)(meta >> 16);
      }
    }
  }
  wave_lds_order();
  // V: chunk 16 (slot / 4) + m holds channels m, m + 16, ... of four slots.  A lane takes four m of one row: the codes of
  // its channels mb are whole halves of consecutive words (one byte when a row has fewer fields than a half).
  if (kind && (rows >> (lane >> 2) & 1)) {
    const Row row = row_of(lane >> 2);
    const int mq = lane & 3, bits = c.bits_of_class[row.cls];
    const BlockGeom g = block_geom(bits, D, c.format);
    uint32_t d[NM];
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) d[mb] = lds.v[lane >> 2][4 * mb + mq];
    uint8_t* const at = (WHOLE ? (uint8_t*)lds.codes : v.arena[row.cls] + ((int64_t)row.pid * H + h) * g.block_bytes + g.v_codes) +
                        (16 * (row.slot >> 2) + 4 * mq) * g.chunk_bytes + 2 * (row.slot & 1);
    const int u = (row.slot >> 1) & 1;
    auto halves = [&](uint32_t a, uint32_t b, int off) {   // bytes of a below bytes of b, one half for each of the four chunks
      const uint32_t h01 = __builtin_amdgcn_perm(b, a, 0x05010400u), h23 = __builtin_amdgcn_perm(b, a, 0x07030602u);
      *(uint16_t*)(at + off) = (uint16_t)h01;
      *(uint16_t*)(at + off + g.chunk_bytes) = (uint16_t)(h01 >> 16);
      *(uint16_t*)(at + off + 2 * g.chunk_bytes) = (uint16_t)h23;
      *(uint16_t*)(at + off + 3 * g.chunk_bytes) = (uint16_t)(h23 >> 16);
    };
    if (bits == 8) {
#pragma unroll
      for (int w = 0; w < NM / 2; ++w) halves(d[2 * w], d[2 * w + 1], 4 * (u * (NM / 2) + w));
    } else if (bits == 4) {
#pragma unroll
      for (int w = 0; w < NM / 4; ++w) halves(d[4 * w] | d[4 * w + 1] << 4, d[4 * w + 2] | d[4 * w + 3] << 4, 4 * (u * (NM / 4) + w));
    } else {
      const uint32_t a = d[0] | d[1] << 2 | d[2] << 4 | d[3] << 6;
      if constexpr (NM == 8) {
        halves(a, d[4] | d[5] << 2 | d[6] << 4 | d[7] << 6, 4 * u);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) at[u + e * g.chunk_bytes] = (uint8_t)(a >> (8 * e));
      }
    }
  }
  wave_lds_order();
  if (WHOLE) {
    for (int w = lane; w < n_codes; w += 64) page_codes[w] = lds.codes[w];
    for (int w = lane; w < n_meta; w += 64) page_meta[w] = lds.meta[w];
    wave_lds_order();   // (the next unit's first stores come behind these loads)
  }
}

// Blocks a compute unit: eight, as many as its LDS holds at head_dim 128, where registers allow (not binary32 rows, nor the binary64 of the paper's formats).  Vector
// instructions are issued in 68 % of the kernel's time and a block starts with a chain of loads, so another wave shows: 37,000 tokens of 16 prompts,
// with the reset, 82.0 us with seven and divisions by the head count, now 80.0; 60 prompts of 4k to 8k tokens 540 and 523.
__host__ __device__ constexpr int bulk_blocks(int in_dtype, bool fp) { return fp ? 6 : (in_dtype == THINKV_F32 ? 6 : 8); }
template <int D, int IN, bool FP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(bulk_blocks(IN, FP)))) void append_place_bulk_kernel(thinkv_view v, int layer, const void* __restrict__ k_new,
                                                                const void* __restrict__ v_new, const int32_t* __restrict__ tok_seq,
                                                                const int32_t* __restrict__ tok_pos,
                                                                const uint8_t* __restrict__ tok_class, int32_t* __restrict__ tok_handle,
                                                                int n_tok, AppendWs ws, int heads_per_block) {
  __shared__ int s_cls[kBulkTokens], s_pid[kBulkTokens], s_slot[kBulkTokens];
  __shared__ NewPage s_new[kBulkTokens];
  __shared__ int s_tok[kBulkTokens][kPage];   // the tokens of the new pages
  __shared__ int s_n_new;
  __shared__ uint32_t s_old;                  // bit t: token t of the block goes to an existing page
  __shared__ UnitLds<D> s_unit[4];
  const thinkv_config& c = v.cfg;
  const int tid = threadIdx.x, i0 = blockIdx.x * kBulkTokens;
  // this block's share of the kv-heads
  const int H = c.n_kv_heads;
  const int h_lo = blockIdx.y * heads_per_block, h_hi = h_lo + heads_per_block < H ? h_lo + heads_per_block : H;
  // ---- places
  if (tid == 0) s_n_new = s_old = 0;
  __syncthreads();
  {
    constexpr int LPT = 256 / kBulkTokens;
    const int u = tid / LPT;
    Place p = {0, 0, 0, 0, 0, 0, 0};
    if (i0 + u < n_tok) p = settle<LPT, true>(v, layer, ws, tok_seq, tok_pos, tok_class, tok_handle, i0 + u, blockIdx.y == 0);
    if (tid % LPT == 0) {
      s_cls[u] = p.cls; s_pid[u] = p.pid; s_slot[u] = p.slot;
      if (p.ok && !p.whole) atomicOr(&s_old, 1u << u);
      if (p.ok && p.whole && p.slot == 0) s_new[atomicAdd(&s_n_new, 1)] = NewPage{i0 + u, p.cls, p.pid, p.cnt, ws.plan[tok_seq[i0 + u]].hi};
    }
  }
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid < 64) update_pools(v, ws);
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n_new = __builtin_amdgcn_readfirstlane(s_n_new), hn = h_hi - h_lo;
  const uint32_t old = __builtin_amdgcn_readfirstlane(s_old);
  for (int q = wave; q < n_new; q += 4) {   // the new pages' tokens: the next of the type, from the first on
    const NewPage np = s_new[q];
    int found = 0;
    auto take = [&](int i, int cl) {   // tokens i + lane, of types cl
      const int t = i + lane;
      const bool is = t < np.end && cl == np.cls;
      const uint64_t all = __ballot(is);
      const int at = found + __popcll(all & ((1ull << lane) - 1ull));
      if (is && at < np.cnt) s_tok[q][at] = t;
      found += __popcll(all);
    };
    take(np.first, tok_class[min(np.first + lane, np.end - 1)]);
    // (beyond the next 64 tokens eight loads at once: the sixteen tokens of a rare type may lie far apart.  32,768 tokens, a second type
    // every 4,000: 164 us with one load at a time, now 123; every 1,000 122 and 112; types in runs of 64 to 192 tokens 115 either way)
    for (int i = np.first + 64; i < np.end && found < np.cnt; i += 512) {
      int cl[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) cl[u] = tok_class[min(i + 64 * u + lane, np.end - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) take(i + 64 * u, cl[u]);
    }
    found = min(found, np.cnt);   // (fewer only if the sequence ids of the call decrease somewhere)
    if (lane == 0) s_new[q].cnt = found;
    wave_lds_order();
    if (blockIdx.y == 0) {
      int pos = lane < found ? tok_pos[s_tok[q][lane]] : -1;
      if (lane < kPage) v.slot_pos[np.cls][(int64_t)np.pid * kPage + lane] = pos;
#pragma unroll
      for (int d = 8; d >= 1; d >>= 1) pos = max(pos, __shfl_xor(pos, d, 64));
      if (lane == 0) atomicMax(&v.page_pos_max[np.cls][np.pid], pos);
    }
  }
  __syncthreads();
  // Units (page, K or V, head) side by side over the waves, whatever the block's head count: the quotient by it is a product with a reciprocal, exact for
  // the few hundred units there are.  (Heads padded to a power of two, for shifts: the waves whose turn a head that is not there was had nothing to do.  16 prompts of
  // 1k to 4k tokens, 5 heads of 128, with the reset, us: divisions 61.7, padded 63.6, now 56.9; in the paper's formats 101.8, 118.8, 98.7.)
  const uint32_t inv = hn == 1 ? 65537u : (hn == 2 ? 32769u : (hn == 3 ? 21846u : 16385u));
  for (int w = wave; w < 2 * n_new * hn; w += 4) {
    const int pair = (int)((uint32_t)w * inv >> 16), q = pair >> 1, kind = pair & 1, h = h_lo + w - pair * hn;   // neighbours in memory side by side
    const int cls = __builtin_amdgcn_readfirstlane(s_new[q].cls), pid = __builtin_amdgcn_readfirstlane(s_new[q].pid);
    const int cnt = __builtin_amdgcn_readfirstlane(s_new[q].cnt);
    place_unit<D, IN, FP, true>(v, kind ? v_new : k_new, kind, h, [&](int r) { return Row{s_tok[q][r], cls, pid, r}; }, (1u << cnt) - 1u, s_unit[wave]);
  }
  if (old)
    for (int w = wave; w < kBulkTokens / kPage * 2 * hn; w += 4) {
      const int t0 = w / (2 * hn) * kPage, kind = w & 1;
      const uint32_t rows = old >> t0 & 0xFFFFu;
      if (rows)
        place_unit<D, IN, FP, false>(v, kind ? v_new : k_new, kind, h_lo + (w >> 1) % hn,
                                     [&](int r) { return Row{i0 + t0 + r, s_cls[t0 + r], s_pid[t0 + r], s_slot[t0 + r]}; }, rows, s_unit[wave]);
    }
}

int launch_append(const thinkv_view& v, int layer, const void* k_new, const void* v_new, const int32_t* tok_seq,
                  const int32_t* tok_pos, const uint8_t* tok_class, int32_t* tok_handle, int n_tok, int in_dtype,
                  void* workspace, hipStream_t st, const int32_t* ev_seq, const int32_t* ev_handle, int n_ev) {
  AppendWs ws = carve(v.cfg, n_tok, workspace);
  const int S = v.cfg.max_seqs;
  if ((int64_t)n_tok > (int64_t)kLongPrompts * S)
    hipLaunchKernelGGL(append_plan_kernel<512>, dim3(S), dim3(512), 0, st, v, layer, tok_seq, tok_class, n_tok, ws, ev_seq, ev_handle, n_ev);
  else
    hipLaunchKernelGGL(append_plan_kernel<256>, dim3(S), dim3(256), 0, st, v, layer, tok_seq, tok_class, n_tok, ws, ev_seq, ev_handle, n_ev);
  const bool small = n_tok <= kBulkFrom;
  const bool aligned = (((uintptr_t)k_new | (uintptr_t)v_new) & 15) == 0;
  if (!small && aligned) {
    // enough blocks to fill the chip: a mid-sized call spreads the kv-heads of its token groups over blocks
    const int H = v.cfg.n_kv_heads, groups = (n_tok + kBulkTokens - 1) / kBulkTokens;
    // (every block of a group settles its places again, so a large call gives each as many heads as it has waves: one head
    // each took 124 us where four took 94, and eight 97: too few blocks to even out)
    int hpb = (int)(((int64_t)H * groups + 4095) / 4096);
    if (hpb > 2) hpb = 4;   // (a block's units are dealt out by a reciprocal for up to four)
    hpb = hpb < 1 ? 1 : (hpb > H ? H : hpb);
    const dim3 grid(groups, (H + hpb - 1) / hpb);
    const bool fp = v.cfg.format == THINKV_FMT_FP;
#define THINKV_BULK(DD, II, FF)                                                                                                   \
  hipLaunchKernelGGL((append_place_bulk_kernel<DD, II, FF>), grid, dim3(256), 0, st, v, layer, k_new, v_new, tok_seq, tok_pos, \
                     tok_class, tok_handle, n_tok, ws, hpb)
#define THINKV_BULK_IN(DD, FF)                                         \
  if (in_dtype == THINKV_F32) THINKV_BULK(DD, THINKV_F32, FF);         \
  else if (in_dtype == THINKV_F16) THINKV_BULK(DD, THINKV_F16, FF);    \
  else THINKV_BULK(DD, THINKV_BF16, FF)
    if (v.cfg.head_dim == 128) {
      if (fp) { THINKV_BULK_IN(128, true); } else { THINKV_BULK_IN(128, false); }
    } else {
      if (fp) { THINKV_BULK_IN(64, true); } else { THINKV_BULK_IN(64, false); }
    }
#undef THINKV_BULK_IN
#undef THINKV_BULK
  } else {
    // A decode-style call (few tokens) spreads the kv-heads of a token over several workgroups so
    // that their load-quantise-store chains run side by side; a bulk call whose rows are not
    // 16-byte aligned keeps one workgroup per token.
    const int H = v.cfg.n_kv_heads, hp = v.cfg.head_dim == 128 ? 1 : 2;
    const int hpb = small ? hp : ((H + hp - 1) / hp) * hp;
    const dim3 grid(n_tok, (H + hpb - 1) / hpb);
    if (v.cfg.head_dim == 128)
      hipLaunchKernelGGL(append_place_kernel<128>, grid, dim3(256), 0, st, v, layer, k_new, v_new, tok_seq, tok_pos,
                         tok_class, tok_handle, n_tok, in_dtype, ws, hpb);
    else
      hipLaunchKernelGGL(append_place_kernel<64>, grid, dim3(256), 0, st, v, layer, k_new, v_new, tok_seq, tok_pos,
                         tok_class, tok_handle, n_tok, in_dtype, ws, hpb);
  }
  return hipGetLastError() == hipSuccess ? THINKV_OK : THINKV_E_HIP;
}

}  // namespace thinkv
