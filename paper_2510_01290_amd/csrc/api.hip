// C ABI entry points: argument checks and kernel dispatch.  No allocation, no synchronisation; the
// only state is what never changes (the device's compute-unit count, the address of the
// library's own scratch array on each device).
#include <cstdlib>
#include "decode_common.h"

namespace thinkv {
size_t append_ws_bytes(const thinkv_config& c, int n_tok);
int launch_append(const thinkv_view& v, int layer, const void* k_new, const void* v_new, const int32_t* tok_seq,
                  const int32_t* tok_pos, const uint8_t* tok_class, int32_t* tok_handle, int n_tok, int in_dtype,
                  void* workspace, hipStream_t st, const int32_t* ev_seq, const int32_t* ev_handle, int n_ev);
int launch_evict(const thinkv_view& v, int layer, const int32_t* ev_seq, const int32_t* ev_handle, int n_ev, hipStream_t st);
int launch_init(const thinkv_view& v, hipStream_t st);
int launch_decode_simple(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
int launch_decode_mfma(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
size_t tbe_ws_bytes(const thinkv_config& c, int n_tok, int n_seg);
size_t tbe_plan_ws_bytes(int B, int max_cuts);
int launch_tbe_plan(const thinkv_view& v, int layer, const int32_t* seq_ids, const int32_t* seg_start, const uint8_t* seg_type,
                    const int32_t* n_segs, const uint8_t* transition_ended, int32_t* seg_count, int rule, int B, int max_segs, int budget, int max_cuts,
                    int cap_seg, int cap_tok, int32_t* tok_seq, int32_t* tok_handle, int32_t* seg_offset, int32_t* seg_keep,
                    int32_t* counts, void* workspace, hipStream_t st);
int launch_tbe_select(const thinkv_view& v, int layer, const int32_t* tok_seq, const int32_t* tok_handle, const int32_t* seg_offset,
                      const int32_t* seg_keep, int n_seg, int n_tok, int max_iters, int32_t* ev_handle, void* workspace,
                      hipStream_t st);
int launch_decode_mfma_stat(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
int launch_stat_fill(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
int launch_stat_count(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
int launch_decode_merge(const thinkv_view& v, const DecodeArgs& a, hipStream_t st);
int decode_mfma_supported(const thinkv_config& c);
int launch_gather_rows(const void* src, void* dst, const int32_t* rows, int64_t n_rows, int row_bytes, int n_wg, hipStream_t st);
int launch_probe_stream(const thinkv_view& v, int layer, const int32_t* seq_ids, int B, int per_head, uint32_t* checksum, hipStream_t st);


static int check_config(const thinkv_config* c) {
  if (!c) return THINKV_E_INVALID_ARG;
  if (c->page_size != kPage || c->group_size != kGroup) return THINKV_E_SHAPE;
  if (c->head_dim != 64 && c->head_dim != 128) return THINKV_E_SHAPE;
  if (c->n_layers < 1 || c->n_kv_heads < 1 || c->n_q_heads < 1 || c->max_seqs < 1 || c->max_pages < 1) return THINKV_E_SHAPE;
  if (c->n_q_heads % c->n_kv_heads) return THINKV_E_SHAPE;
  if (c->n_q_heads / c->n_kv_heads > 8) return THINKV_E_SHAPE;
  if (c->max_pages >= (1 << 24)) return THINKV_E_SHAPE;
  for (int k = 0; k < 3; ++k)
    if (!bits_ok(c->bits_of_class[k])) return THINKV_E_SHAPE;
  if (c->format != THINKV_FMT_INT && c->format != THINKV_FMT_FP) return THINKV_E_UNSUPPORTED;
  if (c->format == THINKV_FMT_FP)
    for (int k = 0; k < 2; ++k)
      if (!(c->fp8_scale[k] > 0.0f) || !(c->fp8_scale[k] < 3.0e38f)) return THINKV_E_INVALID_ARG;
  return THINKV_OK;
}

static int check_view(const thinkv_view* v) {
  if (!v) return THINKV_E_INVALID_ARG;
  int rc = check_config(&v->cfg);
  if (rc) return rc;
  for (int k = 0; k < 3; ++k) {
    if (v->arena_pages[k] < 0 || v->arena_pages[k] > 0x7fffffff) return THINKV_E_INVALID_ARG;
    if (v->arena_pages[k] > 0 && (!v->arena[k] || !v->free_stack[k] || !v->page_filled[k] || !v->slot_pos[k] || !v->page_pos_max[k]))
      return THINKV_E_INVALID_ARG;
  }
  if (!v->free_top || !v->block_table || !v->slot_mask || !v->n_pages || !v->n_live || !v->work_counters || !v->append_counters || !v->dev_status) return THINKV_E_INVALID_ARG;
  return THINKV_OK;
}

// Item sizes of the plain kernel (fast = false: workgroups of four waves, three to a compute unit), and the row counts that the workspace
// is sized for (rows_bound: the most over both kernels, with and without a window).  The fast kernel sizes its launches by
// size_stream and size_window, inside that bound; with fast = true this function only says how many rows a caller has to provide, and
// what callers provide does not change.
// An item pays a fixed price (query set-up, type switches, its partial row), so it is given at least a few page
// pairs.  Where the launch has few (query, kv-head) pairs, the items of the longest sequence fill
// the machine exactly once; where it has many, an item per so many pages, a few rounds of
// them if every sequence were as long as the host's bound.  With a window most pages are merely scanned (a few bytes a page), so
// an item takes more of them.
static int compute_units() {
  static int cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cached[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    cached[dev] = cus;
  }
  return cached[dev];
}

struct ItemSizing {
  int n_rows, per_head, ppi;
};

static ItemSizing size_items(const thinkv_config& c, int B, int max_ctx_pages, int window, bool fast) {
  const int64_t heads = (int64_t)B * c.n_kv_heads;
  const int64_t resident = fast ? (int64_t)compute_units() * 4 * (c.head_dim == 64 ? 3 : 2) : (int64_t)compute_units() * 3;
  const int least = window > 0 ? (fast ? 64 : 256) : (fast ? 16 : 32);   // fewest pages worth an item
  int64_t cap = ((int64_t)max_ctx_pages + least - 1) / least;
  if (cap < 1) cap = 1;
  if (cap > kMaxRowsPerHead) cap = kMaxRowsPerHead;
  int64_t per_head;
  if (window > 0)
    per_head = resident / heads;
  else if (heads * 2 <= resident)
    // all items resident at once; twice as many for larger batches, which are rarely of one length: an item per so many
    // pages then gives the longer contexts more workers than the shorter ones, and late items find what is left
    per_head = (B > 32 ? 2 : 1) * resident / heads;
  else
    per_head = ((fast ? 16 : 4) * resident + heads - 1) / heads;
  if (per_head > cap) per_head = cap;
  if (per_head < 1) per_head = 1;
  ItemSizing z;
  z.per_head = (int)per_head;
  z.n_rows = (int)(per_head * heads);
  z.ppi = (int)(((int64_t)max_ctx_pages + per_head - 1) / per_head);
  if (z.ppi < 1) z.ppi = 1;
  return z;
}

// partial rows any decode call with these bounds can need
static int64_t rows_bound(const thinkv_config& c, int B, int max_ctx_pages) {
  int64_t most = 1;
  for (int fast = 0; fast < 2; ++fast)
    for (int window = 0; window < 2; ++window) {
      const ItemSizing z = size_items(c, B, max_ctx_pages, window, fast != 0);
      if (z.n_rows > most) most = z.n_rows;
    }
  return most;
}

// Full-attention layers of the fast kernel: workgroups of *waves waves.
// Dealt (*grid > 0, deal_item): a workgroup per compute unit, of all the waves it holds, and every item at once; the device sizes
// them by what the sequences hold.  Up to two heads a compute unit, three at head_dim 64; with more, one item a head fills the
// machine, and the short sequences leave it early (96 x 8 heads of 4k..32k tokens, head_dim 128: 350 us dealt, 337 by the
// rule below; head_dim 64, of 16k each: 229 and 246).
// A head to a workgroup, which writes the result itself, where an item would be worth less than the merge launch: contexts of up
// to 96 pages, 352 if every other compute unit has a head, 1,280 with about as many heads as compute units (half as much
// again at head_dim 64, where a page is half the work), 256 with more heads and 512 with more than two a compute unit.
// Measured on both sides, 8 kv-heads of 128, us: 8 x 1k tokens (66 pages) 16.9 so and 17.9 dealt, 8 x 2k 20.9 and 18.4, in the
// paper's formats 29.6 and 23.5; 24 x 3k (200 pages) 29.5 and 32.7, 17 x 8k 56 and 49; 32 x 8k 65.9 and 69.8, 32 x 16k 132 and 138 (but 32 x 3.2k..32k 166 and 114); head_dim 64, 16 x 2 heads
// of 1.5k 16.8 and 20.1.
// More heads: workgroups of four, several to a compute unit, so that one's start and end are covered by the others', and an
// item per so many pages: about sixteen rounds of them if every sequence were as long as the host's bound, but no
// fewer than 128 pages a wave (64 pages: head_dim 64, 64 heads, 96 x 4k tokens 76 us, now 65; 128 x 16k 326, now 307).
static ItemSizing size_stream(const thinkv_config& c, int B, int max_ctx_pages, int* waves, int* grid) {
  const int64_t heads = (int64_t)B * c.n_kv_heads, cus = compute_units();
  const int64_t full = 4 * decode_waves_per_simd(c.head_dim, c.format == THINKV_FMT_FP);
  const int64_t pages = max_ctx_pages > 0 ? max_ctx_pages : 1;
  const int64_t most = (pages + 7) / 8, bound = rows_bound(c, B, max_ctx_pages);   // rows: what the workspace is sized for
  const bool few = heads <= cus;
  const bool single = few ? pages <= (10 * heads >= 9 * cus ? 1280 : (2 * heads > cus ? 352 : 96)) * (c.head_dim == 64 ? 3 : 2) / 2 : pages <= (heads <= 2 * cus ? 256 : 512);
  ItemSizing z;
  *grid = 0;
  if (heads <= (c.head_dim == 64 ? 3 : 2) * cus && B <= kDealSeqs && !single) {
    const int64_t wanted = heads * ((pages + kDealPages * full - 1) / (kDealPages * full));
    *waves = (int)full;
    *grid = (int)(wanted < cus ? wanted : cus);
    z.n_rows = (int)(*grid * full < bound ? *grid * full : bound);
    z.per_head = z.ppi = 1;   // (not used)
    return z;
  }
  const int64_t W = few ? (most < full ? most : full) : (most < 4 ? most : 4);
  int64_t per_head = few ? 1 : (16 * cus * full + heads * W - 1) / (heads * W);
  const int64_t cap = few ? 1 : (pages + 128 * W - 1) / (128 * W), room = bound / heads;   // (room is at least 1)
  if (per_head > cap) per_head = cap;
  if (per_head > room) per_head = room;
  if (per_head > kMaxRowsPerHead) per_head = kMaxRowsPerHead;
  *waves = (int)W;
  z.per_head = (int)per_head;
  z.n_rows = (int)(per_head * heads);
  z.ppi = (int)((pages + per_head - 1) / per_head);
  return z;
}

// Sliding-window layers of the fast kernel: an item is a workgroup of all the waves of a compute unit that scans the page lists for hg kv-heads and
// attends what is visible with an hg-th of its waves a head.  As many heads to a workgroup as leave a workgroup for every compute
// unit (fewer repeated scans), and, where even one head a workgroup does not, several items to a head.  How many follows from the
// two things an item spends its time on.  What is visible: the window's tokens lie in as few pages as hold them, or, where they
// took freed slots, a few to a page all over the lists, so above 512 tokens an item per 128 of them.  2 x 8 heads of 128, 16k tokens, window 1,024, us with an item per 512
// tokens / 256 / 128: a third of the slots reused once 27.3 / 22.9 / 20.5, four times 22.6 / 19.1 / 17.7, heads of 64 23.7 / 20.3 / 18.1; all in fresh pages, where the
// last item has everything, 18.9 / 18.7 / 19.2, and 15.0 with one item a head, which takes 24.7 in reused slots.
// And the scan: above 6,144 pages an item per 2,048 of them (8 x 8 heads of 128, window 128: 131k tokens 23.9 us with one item, 16.8 so,
// 262k 36.9 and 21.8; heads of 64 20.0 and 17.3, 28.6 and 20.0).  An item per 1,024 above 3,072 gains at head_dim 128 (8 x 65k 17.4 and 14.9) and loses the merge launch at 64 (8 x 50k
// 13.4 and 15.8), where a workgroup scans half as many pages again at a time, and with many heads (16 x 56k 16.9 and 18.0).
static ItemSizing size_window(const thinkv_config& c, int B, int max_ctx_pages, int window, int* heads_per_group) {
  const int64_t heads = (int64_t)B * c.n_kv_heads, cus = compute_units();
  int hg = 1;
  while (2 * hg <= window_waves(c.head_dim) && 2 * hg <= c.n_kv_heads && heads >= 2 * hg * cus) hg *= 2;
  const int64_t groups = (int64_t)B * ((c.n_kv_heads + hg - 1) / hg);
  const int64_t pages = max_ctx_pages > 0 ? max_ctx_pages : 1;
  int64_t per_head = cus / groups;
  const int64_t visible = window > 512 ? ((int64_t)window + 127) / 128 : 1, scanned = pages > 6144 ? (pages + 2047) / 2048 : 1;
  const int64_t cap = visible > scanned ? visible : scanned, by_pages = (pages + 63) / 64, room = rows_bound(c, B, max_ctx_pages) / heads;
  if (per_head > cap) per_head = cap;
  if (per_head > by_pages) per_head = by_pages;
  if (per_head > room) per_head = room;
  if (per_head > kMaxRowsPerHead) per_head = kMaxRowsPerHead;
  if (per_head < 1) per_head = 1;
  *heads_per_group = hg;
  ItemSizing z;
  z.per_head = (int)per_head;
  z.n_rows = (int)(per_head * heads);
  z.ppi = (int)((pages + per_head - 1) / per_head);
  return z;
}

static size_t partial_bytes_of(const thinkv_config& c, int64_t rows) {
  const int G = c.n_q_heads / c.n_kv_heads;
  return (size_t)rows * G * (c.head_dim + kRowPad) * sizeof(float);
}

static int decode_common(const thinkv_view* view, int32_t layer, const void* q, void* out, float* lse,
                         const int32_t* seq_ids, const int32_t* q_pos, int32_t B, int32_t window, float softmax_scale,
                         int q_dtype, int out_dtype, int32_t max_ctx_pages, void* workspace, size_t workspace_bytes,
                         void* stream, bool fast, float* sparsity = nullptr) {
  int rc = check_view(view);
  if (rc) return rc;
  if (B < 0 || layer < 0 || layer >= view->cfg.n_layers || window < 0 || max_ctx_pages < 0) return THINKV_E_INVALID_ARG;
  if (B > view->cfg.max_seqs) return THINKV_E_INVALID_ARG;   // at most a query per sequence of the view
  if (!(softmax_scale > 0.0f) || !(softmax_scale < 3.0e38f)) return THINKV_E_INVALID_ARG;   // also rejects NaN
  if (B == 0) return THINKV_OK;
  if (!q || !out || !seq_ids || !workspace || (window > 0 && !q_pos)) return THINKV_E_INVALID_ARG;
  if (q_dtype != THINKV_F16 && q_dtype != THINKV_BF16) return THINKV_E_UNSUPPORTED;
  if (out_dtype != THINKV_F16 && out_dtype != THINKV_BF16 && out_dtype != THINKV_F32) return THINKV_E_UNSUPPORTED;
  fast = fast && decode_mfma_supported(view->cfg);
  if (sparsity && !fast) return THINKV_E_UNSUPPORTED;
  const size_t partial_bytes = thinkv_decode_workspace_bytes(&view->cfg, B, max_ctx_pages);
  if (workspace_bytes < (sparsity ? thinkv_decode_sparsity_workspace_bytes(&view->cfg, B, max_ctx_pages) : partial_bytes)) return THINKV_E_WORKSPACE;
  DecodeArgs a;
  a.q = q;
  a.out = out;
  a.lse = lse;
  a.seq_ids = seq_ids;
  a.q_pos = q_pos;
  a.partial = (float*)workspace;
  a.layer = layer;
  a.B = B;
  a.window = window;
  a.q_dtype = q_dtype;
  a.out_dtype = out_dtype;
  a.waves = a.grid = 0;
  const ItemSizing z = !fast ? size_items(view->cfg, B, max_ctx_pages, window, false)
                             : (window > 0 ? size_window(view->cfg, B, max_ctx_pages, window, &a.waves) : size_stream(view->cfg, B, max_ctx_pages, &a.waves, &a.grid));
  if (z.n_rows > rows_bound(view->cfg, B, max_ctx_pages)) return THINKV_E_WORKSPACE;   // cannot happen: a launch never has more rows than the workspace
  a.n_rows = z.n_rows;
  a.per_head = z.per_head;
  a.ppi = z.ppi;
  // the heads' first rows and row counts behind the partial rows
  a.alloc = (int32_t*)((char*)workspace + ((partial_bytes_of(view->cfg, rows_bound(view->cfg, B, max_ctx_pages)) + 255) & ~(size_t)255));
  a.scale_log2e = softmax_scale * 1.4426950408889634f;
  a.stat = nullptr;
  a.stat_stride = 0;
  a.sparsity = sparsity;
  a.stat_sum = nullptr;
  a.direct = fast && !sparsity && !a.grid && a.per_head == 1;   // short contexts or huge batches: one item per head, no merge launch
  hipStream_t st = (hipStream_t)stream;
  if (sparsity) {
    // pooled scores behind the partials (whose size is a multiple of 16 bytes)
    a.stat = (float*)((char*)workspace + ((partial_bytes + 255) & ~(size_t)255));
    a.stat_stride = (int64_t)kPage * (max_ctx_pages > 0 ? max_ctx_pages : 1);
    // Behind the pooled scores, where there is a word of four bytes for every head: a word of eight for every query, if it can be one
    // (a workspace need not be aligned), holds the sum of that many heads, and all counting workgroups, two to a compute unit, are there
    // at once.  With more of them what each waits for its addition adds up: us by a launch of its own for the mean / by sums: 1 x 2k tokens 21.6 / 20.4, 16 x 8k..32k
    // 97.7 / 96.7, 64 x 1k..10k 70.3 / 70.0, 256 x 1k 126.8 / 127.6.
    unsigned long long* const sum = (unsigned long long*)(a.stat + (int64_t)B * view->cfg.n_kv_heads * a.stat_stride);
    const int64_t heads = (int64_t)B * view->cfg.n_kv_heads;
    if (view->cfg.n_kv_heads >= 2 && view->cfg.n_kv_heads <= kStatHeads && heads <= 2 * compute_units() && ((uintptr_t)sum & 7) == 0) a.stat_sum = sum;
    rc = launch_stat_fill(*view, a, st);
    if (rc) return rc;
    rc = launch_decode_mfma_stat(*view, a, st);
    if (rc) return rc;
    return launch_stat_count(*view, a, st);   // and the merge
  }
  rc = fast ? launch_decode_mfma(*view, a, st) : launch_decode_simple(*view, a, st);
  if (rc || a.direct) return rc;
  return launch_decode_merge(*view, a, st);
}

}  // namespace thinkv

using namespace thinkv;

extern "C" {

size_t thinkv_block_bytes(const thinkv_config* cfg, int bits) {
  if (check_config(cfg) || !bits_ok(bits)) return 0;
  return (size_t)block_geom(bits, cfg->head_dim, cfg->format).block_bytes;
}

size_t thinkv_page_bytes(const thinkv_config* cfg, int bits) {
  return thinkv_block_bytes(cfg, bits) * (cfg ? (size_t)cfg->n_kv_heads : 0);
}

size_t thinkv_append_workspace_bytes(const thinkv_config* cfg, int32_t n_tok) {
  if (check_config(cfg) || n_tok < 0) return 0;
  return append_ws_bytes(*cfg, n_tok);
}

size_t thinkv_decode_workspace_bytes(const thinkv_config* cfg, int32_t B, int32_t max_ctx_pages) {
  if (check_config(cfg) || B < 0 || max_ctx_pages < 0) return 0;
  // partial rows, then two words per (query, kv-head)
  const int b1 = B > 0 ? B : 1;
  return ((partial_bytes_of(*cfg, rows_bound(*cfg, b1, max_ctx_pages)) + 255) & ~(size_t)255) + (size_t)b1 * cfg->n_kv_heads * 2 * sizeof(int32_t) + 256;
}

size_t thinkv_decode_sparsity_workspace_bytes(const thinkv_config* cfg, int32_t B, int32_t max_ctx_pages) {
  const size_t partial = thinkv_decode_workspace_bytes(cfg, B, max_ctx_pages);
  if (partial == 0) return 0;
  return ((partial + 255) & ~(size_t)255) +
         (size_t)(B > 0 ? B : 1) * cfg->n_kv_heads * (kPage * (size_t)(max_ctx_pages > 0 ? max_ctx_pages : 1) + 1) * sizeof(float);
}

int thinkv_init_view(const thinkv_view* view, void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  return launch_init(*view, (hipStream_t)stream);
}

int thinkv_append_quantized(const thinkv_view* view, int32_t layer, const void* k_new, const void* v_new,
                            const int32_t* tok_seq, const int32_t* tok_pos, const uint8_t* tok_class,
                            int32_t* tok_handle, int32_t n_tok, thinkv_dtype in_dtype, void* workspace,
                            size_t workspace_bytes, void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  if (n_tok < 0 || layer < 0 || layer >= view->cfg.n_layers) return THINKV_E_INVALID_ARG;
  if (n_tok == 0) return THINKV_OK;
  if (!k_new || !v_new || !tok_seq || !tok_pos || !tok_class || !workspace) return THINKV_E_INVALID_ARG;
  if (in_dtype != THINKV_F16 && in_dtype != THINKV_BF16 && in_dtype != THINKV_F32) return THINKV_E_UNSUPPORTED;
  if (workspace_bytes < append_ws_bytes(view->cfg, n_tok)) return THINKV_E_WORKSPACE;
  return launch_append(*view, layer, k_new, v_new, tok_seq, tok_pos, tok_class, tok_handle, n_tok, (int)in_dtype,
                       workspace, (hipStream_t)stream, nullptr, nullptr, 0);
}

int thinkv_evict_append(const thinkv_view* view, int32_t layer, const int32_t* ev_seq, const int32_t* ev_handle, int32_t n_ev,
                        const void* k_new, const void* v_new, const int32_t* tok_seq, const int32_t* tok_pos,
                        const uint8_t* tok_class, int32_t* tok_handle, int32_t n_tok, thinkv_dtype in_dtype, void* workspace,
                        size_t workspace_bytes, void* stream) {
  // a long eviction list (every plan workgroup reads all of it: one workgroup per sequence slot of the view), or no
  // tokens to append: the two calls one after the other
  if (n_tok <= 0 || n_ev <= 0 || n_ev > 4096 || (view && (int64_t)n_ev * view->cfg.max_seqs > (1 << 20))) {
    const int rc = thinkv_evict(view, layer, ev_seq, ev_handle, n_ev, stream);
    if (rc) return rc;
    return thinkv_append_quantized(view, layer, k_new, v_new, tok_seq, tok_pos, tok_class, tok_handle, n_tok, in_dtype, workspace,
                                   workspace_bytes, stream);
  }
  int rc = check_view(view);
  if (rc) return rc;
  if (layer < 0 || layer >= view->cfg.n_layers) return THINKV_E_INVALID_ARG;
  if (!ev_seq || !ev_handle || !k_new || !v_new || !tok_seq || !tok_pos || !tok_class || !workspace) return THINKV_E_INVALID_ARG;
  if (in_dtype != THINKV_F16 && in_dtype != THINKV_BF16 && in_dtype != THINKV_F32) return THINKV_E_UNSUPPORTED;
  if (workspace_bytes < append_ws_bytes(view->cfg, n_tok)) return THINKV_E_WORKSPACE;
  return launch_append(*view, layer, k_new, v_new, tok_seq, tok_pos, tok_class, tok_handle, n_tok, (int)in_dtype, workspace,
                       (hipStream_t)stream, ev_seq, ev_handle, n_ev);
}

int thinkv_evict(const thinkv_view* view, int32_t layer, const int32_t* ev_seq, const int32_t* ev_handle, int32_t n_ev,
                 void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  if (n_ev < 0 || layer < 0 || layer >= view->cfg.n_layers) return THINKV_E_INVALID_ARG;
  if (n_ev == 0) return THINKV_OK;
  if (!ev_seq || !ev_handle) return THINKV_E_INVALID_ARG;
  return launch_evict(*view, layer, ev_seq, ev_handle, n_ev, (hipStream_t)stream);
}

int thinkv_decode_attention(const thinkv_view* view, int32_t layer, const void* q, void* out, float* lse,
                            const int32_t* seq_ids, const int32_t* q_pos, int32_t B, int32_t window,
                            float softmax_scale, thinkv_dtype q_dtype, thinkv_dtype out_dtype, int32_t max_ctx_pages,
                            void* workspace, size_t workspace_bytes, void* stream) {
  return decode_common(view, layer, q, out, lse, seq_ids, q_pos, B, window, softmax_scale, (int)q_dtype, (int)out_dtype,
                       max_ctx_pages, workspace, workspace_bytes, stream, true);
}

// Partial rows of thinkv_decode_attention_noalloc.  In host code this name is only a stand-in for the
// symbol: the array's address on a device comes from hipGetSymbolAddress (once per device, below).
static __device__ __align__(256) unsigned char scratch[THINKV_NOALLOC_SCRATCH_BYTES];

int thinkv_decode_attention_noalloc(const thinkv_view* view, int32_t layer, const void* q, void* out, float* lse,
                                    const int32_t* seq_ids, const int32_t* q_pos, int32_t B, int32_t window,
                                    float softmax_scale, thinkv_dtype q_dtype, thinkv_dtype out_dtype,
                                    int32_t max_ctx_pages, void* stream) {
  static void* scratch_of_device[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return THINKV_E_HIP;
  if (scratch_of_device[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return THINKV_E_HIP;
    scratch_of_device[dev] = p;
  }
  if (view && B > 0 && max_ctx_pages >= 0 && check_config(&view->cfg) == THINKV_OK &&
      thinkv_decode_workspace_bytes(&view->cfg, B, max_ctx_pages) > (size_t)THINKV_NOALLOC_SCRATCH_BYTES)
    return THINKV_E_WORKSPACE;
  return decode_common(view, layer, q, out, lse, seq_ids, q_pos, B, window, softmax_scale, (int)q_dtype, (int)out_dtype,
                       max_ctx_pages, scratch_of_device[dev], (size_t)THINKV_NOALLOC_SCRATCH_BYTES, stream, true);
}

int thinkv_decode_attention_valu(const thinkv_view* view, int32_t layer, const void* q, void* out, float* lse,
                                 const int32_t* seq_ids, const int32_t* q_pos, int32_t B, int32_t window,
                                 float softmax_scale, thinkv_dtype q_dtype, thinkv_dtype out_dtype, int32_t max_ctx_pages,
                                 void* workspace, size_t workspace_bytes, void* stream) {
  return decode_common(view, layer, q, out, lse, seq_ids, q_pos, B, window, softmax_scale, (int)q_dtype, (int)out_dtype,
                       max_ctx_pages, workspace, workspace_bytes, stream, false);
}

int thinkv_decode_attention_sparsity(const thinkv_view* view, int32_t layer, const void* q, void* out, float* lse,
                                     float* sparsity, const int32_t* seq_ids, const int32_t* q_pos, int32_t B,
                                     int32_t window, float softmax_scale, thinkv_dtype q_dtype, thinkv_dtype out_dtype,
                                     int32_t max_ctx_pages, void* workspace, size_t workspace_bytes, void* stream) {
  if (!sparsity && B > 0) return THINKV_E_INVALID_ARG;
  return decode_common(view, layer, q, out, lse, seq_ids, q_pos, B, window, softmax_scale, (int)q_dtype, (int)out_dtype,
                       max_ctx_pages, workspace, workspace_bytes, stream, true, sparsity);
}

size_t thinkv_tbe_workspace_bytes(const thinkv_config* cfg, int32_t n_tok, int32_t n_seg) {
  if (check_config(cfg) || n_tok < 0 || n_seg < 0) return 0;
  return tbe_ws_bytes(*cfg, n_tok, n_seg);
}

int thinkv_tbe_select(const thinkv_view* view, int32_t layer, const int32_t* tok_seq, const int32_t* tok_handle,
                      const int32_t* seg_offset, const int32_t* seg_keep, int32_t n_seg, int32_t n_tok,
                      int32_t max_iters, int32_t* ev_handle, void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  if (n_seg < 0 || n_tok < 0 || max_iters < 1 || layer < 0 || layer >= view->cfg.n_layers) return THINKV_E_INVALID_ARG;
  if (n_seg == 0 || n_tok == 0) return THINKV_OK;
  if (!tok_seq || !tok_handle || !seg_offset || !seg_keep || !ev_handle || !workspace) return THINKV_E_INVALID_ARG;
  if (workspace_bytes < tbe_ws_bytes(view->cfg, n_tok, n_seg)) return THINKV_E_WORKSPACE;
  return launch_tbe_select(*view, layer, tok_seq, tok_handle, seg_offset, seg_keep, n_seg, n_tok, max_iters, ev_handle,
                           workspace, (hipStream_t)stream);
}

size_t thinkv_tbe_plan_workspace_bytes(int32_t B, int32_t max_cuts) {
  if (B < 0 || max_cuts < 1) return 0;
  return tbe_plan_ws_bytes(B, max_cuts);
}

int thinkv_tbe_plan(const thinkv_view* view, int32_t layer, const int32_t* seq_ids, const int32_t* seg_start,
                    const uint8_t* seg_type, const int32_t* n_segs, const uint8_t* transition_ended, int32_t* seg_count, int32_t rule, int32_t B,
                    int32_t max_segs, int32_t budget, int32_t max_cuts, int32_t cap_seg, int32_t cap_tok,
                    int32_t* tok_seq, int32_t* tok_handle, int32_t* seg_offset, int32_t* seg_keep, int32_t* counts,
                    void* workspace, size_t workspace_bytes, void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  if (B < 0 || layer < 0 || layer >= view->cfg.n_layers || budget < 0 || cap_seg < 0 || cap_tok < 0) return THINKV_E_INVALID_ARG;
  if (max_segs < 1 || max_segs > THINKV_TBE_MAX_SEGS || max_cuts < 1 || max_cuts > THINKV_TBE_MAX_SEGMENT) return THINKV_E_INVALID_ARG;
  if (!seq_ids || !seg_start || !seg_type || !n_segs || !tok_seq || !tok_handle || !seg_offset || !seg_keep || !counts || !workspace)
    return THINKV_E_INVALID_ARG;
  if (rule != THINKV_TBE_BY_COUNT && rule != THINKV_TBE_BY_SIZE) return THINKV_E_INVALID_ARG;
  if (rule == THINKV_TBE_BY_COUNT && !seg_count) return THINKV_E_INVALID_ARG;
  if (workspace_bytes < tbe_plan_ws_bytes(B, max_cuts)) return THINKV_E_WORKSPACE;
  return launch_tbe_plan(*view, layer, seq_ids, seg_start, seg_type, n_segs, transition_ended, seg_count, rule, B, max_segs, budget, max_cuts,
                         cap_seg, cap_tok, tok_seq, tok_handle, seg_offset, seg_keep, counts, workspace, (hipStream_t)stream);
}

int thinkv_probe_stream_pages(const thinkv_view* view, int32_t layer, const int32_t* seq_ids, int32_t B, uint32_t* checksum, void* stream) {
  int rc = check_view(view);
  if (rc) return rc;
  if (B < 0 || layer < 0 || layer >= view->cfg.n_layers || B > view->cfg.max_seqs) return THINKV_E_INVALID_ARG;
  if (B == 0) return THINKV_OK;
  if (!seq_ids || !checksum) return THINKV_E_INVALID_ARG;
  // four waves to a workgroup, as many workgroups as fill the machine at the occupancy of the attention kernel
  int64_t per_head = (int64_t)compute_units() * (view->cfg.head_dim == 64 ? 3 : 2) / ((int64_t)B * view->cfg.n_kv_heads);
  if (per_head < 1) per_head = 1;
  return launch_probe_stream(*view, layer, seq_ids, B, (int)per_head, checksum, (hipStream_t)stream);
}

int thinkv_gather_rows(const void* src, void* dst, const int32_t* rows, int64_t n_rows, int32_t row_bytes, void* stream) {
  if (n_rows < 0 || row_bytes <= 0 || row_bytes % 16) return THINKV_E_INVALID_ARG;
  if (n_rows == 0) return THINKV_OK;
  if (!src || !dst || !rows) return THINKV_E_INVALID_ARG;
  if (((uintptr_t)src | (uintptr_t)dst) & 15) return THINKV_E_INVALID_ARG;
  const int64_t pieces = n_rows * (row_bytes / 16);
  int64_t n_wg = (pieces + 1023) / 1024;                      // four pieces a thread
  const int64_t most = (int64_t)compute_units() * 16;        // a few rounds of workgroups at most: the loop does the rest
  if (n_wg > most) n_wg = most;
  return launch_gather_rows(src, dst, rows, n_rows, row_bytes, (int)n_wg, (hipStream_t)stream);
}

const char* thinkv_status_string(int status) {
  switch (status) {
    case THINKV_OK: return "ok";
    case THINKV_E_INVALID_ARG: return "invalid argument";
    case THINKV_E_SHAPE: return "unsupported geometry";
    case THINKV_E_UNSUPPORTED: return "unsupported dtype or option";
    case THINKV_E_WORKSPACE: return "workspace too small";
    case THINKV_E_HIP: return "HIP call failed";
  }
  return "unknown status";
}

}  // extern "C"
