"""Decode attention at the edges of its work distribution: items of one and of several workgroups, short lists, a
ring that wraps, pages with nothing live, batches whose row count is limited by the workspace, and value scales that leave
the range of the second matrix operand.  The reference is the plain vector-ALU kernel (itself checked against the oracle);
the workspace has exactly the size the library asks for, with a guard behind it."""
import numpy as np
import pytest
import torch

from paper_2510_01290_amd import binding as B

pytestmark = pytest.mark.gpu


def _cache(D, G, H, ctx, fmt, bits, seed, v_scale=1.0, dead=0.0):
    """a cache of len(ctx) sequences, types in runs of 1..60 tokens; a share `dead` of the runs is evicted as a whole"""
    rng = np.random.default_rng(seed)
    S, n = len(ctx), int(np.sum(ctx))
    seq = np.repeat(np.arange(S), ctx).astype(np.int32)
    pos = np.concatenate([np.arange(c) for c in ctx]).astype(np.int32)
    runs = np.repeat(np.arange(n), rng.integers(1, 61, n))[:n]
    cls = rng.integers(0, 3, n).astype(np.uint8)[runs]
    most = int(max(ctx)) // 16 + 3
    c = B.Cache(1, G * H, H, D, bits, S, most, [n // 16 + 3 * S + 8] * 3, fmt=fmt, fp8_scale=(0.05, 0.05 * v_scale))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    k = torch.randn((n, H, D), generator=gen, device="cuda:0").to(torch.bfloat16)
    v = (torch.randn((n, H, D), generator=gen, device="cuda:0") * v_scale).to(torch.bfloat16)
    h = torch.empty(n, dtype=torch.int32, device="cuda:0")
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")  # noqa: E731
    B.thinkv_append_quantized(c, 0, k, v, d(seq), d(pos), d(cls), h)
    gone = (rng.random(n) < dead)[runs]
    if gone.any():
        at = d(np.flatnonzero(gone))
        B.thinkv_evict(c, 0, d(seq)[at], h[at])
    q = torch.randn((S, G * H, D), generator=gen, device="cuda:0").to(torch.bfloat16)
    return c, q


def _items(c, ws, need, S):
    """how many items every (query, kv-head) got and where its partial rows begin, as the call left them in its workspace"""
    H = c.cfg.n_kv_heads
    at = need - 256 - 8 * S * H
    alloc = ws[at:at + 8 * S * H].view(torch.int32).view(S, H, 2).cpu()
    return alloc[..., 1], alloc[..., 0]


def _both(c, q, D, bound=None, window=0, q_pos=None, ids=None, items=None):
    S, Hq = q.shape[:2]
    ids = torch.arange(S, dtype=torch.int32, device="cuda:0") if ids is None else torch.tensor(ids, dtype=torch.int32, device="cuda:0")
    pages = int(c.n_pages[:, 0].sum(-1).max()) if bound is None else bound
    qp = None if q_pos is None else torch.tensor(q_pos, dtype=torch.int32, device="cuda:0")
    res = []
    for fn in (B.load().thinkv_decode_attention, B.load().thinkv_decode_attention_valu):
        need = B.thinkv_decode_workspace_bytes(c.cfg, S, pages)
        ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda:0")
        out = torch.empty((S, Hq, D), dtype=torch.float32, device="cuda:0")
        lse = torch.empty((S, Hq), dtype=torch.float32, device="cuda:0")
        rc = fn(B.C.byref(c.view), 0, B._ptr(q), B._ptr(out), B._ptr(lse), B._ptr(ids), B._ptr(qp), S, window, D ** -0.5, B.BF16, B.F32, pages,
                B._ptr(ws), need, B._stream(None))
        torch.cuda.synchronize()
        assert rc == 0
        assert bool((ws[need:] == 0x5A).all()), "written behind the workspace"
        if items is not None and not res:
            items.extend(_items(c, ws, need, S))
        res.append((out.double().cpu(), lse.double().cpu()))
    assert int(c.dev_status.abs().sum()) == 0
    return res


def _close(o, l, ro, rl, least=1.2e-6):
    """Every sequence's outputs to 2e-5 of its own largest one: products whose second operand holds 22 bits are 2e-7 off, and with 11
    bits, one term of the pair lost, 2e-4.  Below that stands what the sums themselves lose: codes and zero-points are summed
    apart, about 4 each for values of N(0, 1), with a rounding of 2^-25 of that for each of some hundred additions a wave and item,
    1.2e-7 * sqrt(100) = 1.2e-6; the largest output of 56,000 tokens is 0.027, so that a lost term would still be seen (6e-6)."""
    for b in range(len(o)):
        fin = torch.isfinite(rl[b])
        assert torch.equal(torch.isfinite(l[b]), fin) and (not fin.any() or float((l[b][fin] - rl[b][fin]).abs().max()) <= 2e-5 * max(1.0, float(rl[b][fin].abs().max())))
        far, top = float((o[b] - ro[b]).abs().max()), float(ro[b].abs().max())
        assert far <= max(2e-5 * top, least), (b, far, top)


@pytest.mark.parametrize("D,G,H,ctx,fmt,bits,dead", [
    (128, 4, 1, [9000], 0, (8, 2, 4), 0.0),                    # several items a head, every ring wraps
    (64, 8, 2, [12000, 1], 0, (8, 4, 2), 0.3),                 # ... and runs of whole pages with nothing live
    (128, 8, 2, [2000, 33, 16, 17, 15, 1], 0, (2, 2, 2), 0.0),  # list lengths around a page, a pair, a chunk
    (64, 1, 3, [700, 129, 128, 127, 256, 8], 0, (8, 8, 8), 0.2),
    (128, 4, 1, [9000], 1, (2, 4, 8), 0.0),
    (64, 8, 2, [5000, 40, 1], 1, (8, 2, 4), 0.3),
    (64, 8, 8, [700] * 127 + [56000], 0, (8, 2, 4), 0.0),      # more heads than are dealt: six items for the longest, as the workspace allows
    (64, 8, 16, [900] * 69 + [30000], 1, (4, 4, 4), 0.0),      # ... in the paper's formats
    (128, 4, 8, [300] * 66 + [20000], 0, (8, 2, 4), 0.1),
    (64, 8, 8, [1500] * 128, 0, (8, 2, 4), 0.0),               # ... of one item each
    (128, 4, 8, [300] * 40, 0, (8, 2, 4), 0.5),
    (128, 4, 8, [2300 + 25 * i for i in range(24)], 0, (8, 2, 4), 0.1),   # a workgroup a head, 150 to 190 pages: chunks of one pair and of four
    (128, 5, 8, [700 + 2100 * (i % 5) for i in range(19)], 0, (8, 2, 4), 0.0),   # ... dealt, several items to a workgroup and several to a head
], ids=lambda x: str(x)[:24].replace(" ", ""))
def test_stream_kernel_against_the_plain_kernel(D, G, H, ctx, fmt, bits, dead):
    print("stream:", D, G, H, len(ctx), max(ctx), fmt, bits, dead, flush=True)
    c, q = _cache(D, G, H, ctx, fmt, bits, 11 + D + G + len(ctx), dead=dead)
    items = []
    (o, l), (ro, rl) = _both(c, q, D, items=items)
    if max(ctx) >= 20000:
        assert int(items[0][-1, 0]) == {56000: 6, 30000: 4, 20000: 3}[max(ctx)] and int(items[0][0, 0]) == 1
    _close(o, l, ro, rl)


@pytest.mark.parametrize("bound", [0, 1, 40, 100000])
def test_stream_kernel_with_a_wrong_context_bound(bound):
    """the host's bound sizes the launch only: too small or far too large, every page is attended"""
    print("stream bound:", bound, flush=True)
    c, q = _cache(128, 4, 2, [1300, 200, 77], 0, (8, 2, 4), 5)
    (o, l), (ro, rl) = _both(c, q, 128, bound)
    _close(o, l, ro, rl)


@pytest.mark.parametrize("D,G,v_scale", [(128, 4, 60.0), (64, 8, 60.0), (128, 8, 3000.0), (64, 4, 8000.0)])
def test_value_scales_out_of_the_lifted_range(D, G, v_scale):
    """value ranges of a few hundred (the softmax reference has to move before the lifted product fits) and of tens of
    thousands (the lift itself is dropped)"""
    print("stream scales:", D, G, v_scale, flush=True)
    c, q = _cache(D, G, 2, [3000, 50], 0, (8, 2, 4), 9, v_scale=v_scale)
    (o, l), (ro, rl) = _both(c, q, D)
    # without the lift, weights below 2^-24 of the largest are lost: 3,000 of them are 2e-4 of the largest value
    assert float((o - ro).abs().max()) <= 5e-4 * float(ro.abs().max())
    assert float((l - rl).abs().max()) <= 1e-4


@pytest.mark.parametrize("D,G,H,ctx,fmt,window,dead", [
    (64, 8, 8, [3000] * 70, 0, 128, 0.3),            # two heads to a workgroup
    (128, 4, 5, [9000, 40, 1, 700], 0, 1024, 0.2),   # one head to a workgroup, several items a head; heads no power of two
    (128, 8, 3, [26000], 0, 30000, 0.0),             # everything visible, many items
    (128, 4, 2, [29000], 0, 400, 0.2),               # lists longer than one scan by one item
    (64, 4, 1, [30000, 500], 1, 900, 0.0),           # a wide window by several items
    (64, 2, 16, [500] * 64, 1, 100, 0.0),
    (128, 4, 8, [17, 16, 300], 1, 1, 0.0),
], ids=lambda x: str(x)[:24].replace(" ", ""))
def test_window_kernel_against_the_plain_kernel(D, G, H, ctx, fmt, window, dead):
    print("window:", D, G, H, len(ctx), max(ctx), fmt, window, dead, flush=True)
    c, q = _cache(D, G, H, ctx, fmt, (8, 2, 4), 21 + D + G + len(ctx), dead=dead)
    items = []
    q_pos = [x - 1 for x in ctx]
    pages = c.block_table[0, 0, 0].long()
    if window == 400:     # a query in the middle: its window reaches over the 512th page of a list
        q_pos = [int(c.slot_pos[0][pages[512]].min()) + 150]
    (o, l), (ro, rl) = _both(c, q, D, window=window, q_pos=q_pos, items=items)
    if window == 900:     # a long scan and a wide window, by several workgroups a head
        assert int(items[0][0, 0]) >= 8
    if window == 400:     # one workgroup a head, which writes the result itself; it scans 512 pages at a time and finds some in two passes
        assert int(items[0][0, 0]) == 0x5A5A5A5A
        seen = c.slot_pos[0][pages[:int(c.n_pages[0, 0, 0])]]
        seen = ((seen <= q_pos[0]) & (seen > q_pos[0] - window)).any(-1)
        assert bool(seen[:512].any()) and bool(seen[512:].any())
    _close(o, l, ro, rl)


def _put(x, t=np.int32):
    return torch.from_numpy(np.ascontiguousarray(x).astype(t)).to("cuda:0")


def _live(c, b, k):
    """[pages, 16] of sequence b, type k: which slots are live, and their positions"""
    n = int(c.n_pages[b, 0, k])
    mask, ids = c.slot_mask[b, 0, k, :n].cpu().numpy(), c.block_table[b, 0, k, :n].long()
    return ((mask[:, None] >> np.arange(16)) & 1).astype(bool), c.slot_pos[k][ids].cpu().numpy()


def _reuse(c, ctx, rng, share, fresh=0.0):
    """evicts a share of the tokens, one by one, and puts new ones into all but `fresh` of their slots: the sequences' last positions"""
    H, D = c.cfg.n_kv_heads, c.cfg.head_dim
    ev_seq, ev_h, cls = [], [], []
    for b in range(len(ctx)):
        for k in range(3):
            live = _live(c, b, k)[0].reshape(-1)
            at = np.flatnonzero(live & (rng.random(len(live)) < share))
            ev_seq.append(np.full(len(at), b))
            ev_h.append(k << 28 | at)               # list index << 4 | slot
            cls.append(np.full(len(at), k))
    seq, h, cls = np.concatenate(ev_seq), np.concatenate(ev_h), np.concatenate(cls)
    B.thinkv_evict(c, 0, _put(seq), _put(h))
    take = rng.random(len(seq)) >= fresh
    order = np.lexsort((rng.random(int(take.sum())), seq[take]))
    seq, cls = seq[take][order], cls[take][order]
    new = np.bincount(seq, minlength=len(ctx))
    pos = np.concatenate([x + np.arange(n) for x, n in zip(ctx, new)])
    if len(seq):
        kv = [torch.randn((len(seq), H, D), device="cuda:0").to(torch.bfloat16) for _ in range(2)]
        B.thinkv_append_quantized(c, 0, kv[0], kv[1], _put(seq), _put(pos), _put(cls, np.uint8))
    return [int(x + n - 1) for x, n in zip(ctx, new)]


@pytest.mark.parametrize("D,G,H,ctx,bits,window,fresh", [
    (64, 8, 8, [3000] * 40 + [5, 17], (8, 2, 4), 128, 0.0),   # a few tokens to a page, a head to a workgroup
    (64, 4, 3, [20000, 33], (2, 4, 8), 30000, 0.0),           # all of it: twenty items a head, tails of less than a pair
    (128, 4, 2, [26000, 1], (4, 8, 2), 30000, 0.0),
    (128, 8, 2, [9000, 800], (8, 2, 4), 700, 0.0),
    (128, 2, 1, [2000], (2, 2, 8), 37, 0.5),                  # some of the freed slots taken
    (64, 1, 16, [400] * 70, (4, 8, 2), 1, 0.0),
], ids=lambda x: str(x)[:24].replace(" ", ""))
def test_window_over_reused_slots(D, G, H, ctx, bits, window, fresh):
    """tokens evicted one by one and their slots taken again: the window's tokens are scattered over the lists.  Against the plain kernel; the
    statistic against full attention's where everything is visible"""
    print("window, reused slots:", D, G, H, len(ctx), max(ctx), bits, window, flush=True)
    c, q = _cache(D, G, H, ctx, 0, bits, 31 + D + G)
    q_pos = _reuse(c, ctx, np.random.default_rng(D + G + window), 0.3, fresh)
    (o, l), (ro, rl) = _both(c, q, D, window=window, q_pos=q_pos)
    _close(o, l, ro, rl)
    if window < max(q_pos):
        return
    S, pages = q.shape[0], int(c.n_pages[:, 0].sum(-1).max())
    ids, qp = torch.arange(S, dtype=torch.int32, device="cuda:0"), _put(q_pos)
    out, sp = torch.empty((S, G * H, D), dtype=torch.float32, device="cuda:0"), [torch.empty(S, dtype=torch.float32, device="cuda:0") for _ in range(2)]
    for w, x in zip((0, window), sp):
        B.thinkv_decode_attention_sparsity(c, 0, q, out, None, x, ids, qp, w, D ** -0.5, pages)
    # (scores alike up to the order of a few additions: one entry in a thousand may change sides)
    assert float((sp[0] - sp[1]).abs().max()) <= 1e-3 and float(sp[0].max()) > 0.01


LIST = 1024   # entries of a type's list of what is visible


def _grouping(c, S):
    """heads of a workgroup, and waves of it"""
    cus, H, waves = torch.cuda.get_device_properties(0).multi_processor_count, c.cfg.n_kv_heads, 8 if c.cfg.head_dim == 128 else 12
    hg = 1
    while 2 * hg <= min(waves, H) and S * H >= 2 * hg * cus:
        hg *= 2
    return hg, waves


def _visible(c, b, q_pos, window, waves, hg):
    """what one item finds for sequence b: entries of each type, whether they are pages, and entries of the first block of the scan"""
    pages, quads = [], []
    for k in range(3):
        live, pos = _live(c, b, k)
        see = live & (pos <= q_pos) & (pos > q_pos - window)
        pages.append(see.any(1).astype(int))
        quads.append(see.reshape(-1, 4, 4).any(2).sum(1))
    block, at = 64 * waves, 0
    while at + block < max(map(len, pages)) and not any(x[at:at + block].any() for x in pages):
        at += block
    first = lambda lists: sum(int(x[at:at + block].sum()) for x in lists)  # noqa: E731
    whole, four = (first(pages) + 1) // 2, (first(quads) + 7) // 8
    by_page = c.cfg.format == B.FMT_FP or whole <= max(waves // hg, four + four // 8 + 1)
    use = pages if by_page else quads
    return [int(x.sum()) for x in use], by_page, [int(x[at:at + block].sum()) for x in use]


MANY = [5] * 15 + [1]   # with 8 kv-heads: an item a head, whatever the others' lengths
@pytest.mark.parametrize("D,G,H,ctx,fmt,bits,window,share,hg,by_page,overflow", [
    (64, 4, 8, [22000] + MANY, 0, (8, 2, 4), -1, 0.3, 1, False, "first"),       # the refilled tokens: the first block of pages has more quads than a list holds
    (128, 5, 8, [33000] + MANY, 0, (2, 4, 8), -1, 0.15, 1, False, "later"),     # ... the second has
    (64, 8, 8, [60000] + MANY, 0, (8, 4, 2), 1 << 20, 0.0, 1, True, "later"),   # whole pages, everything visible
    (128, 8, 8, [54000] + MANY, 0, (8, 2, 4), 1 << 20, 0.05, 1, True, "later"),
    (64, 8, 8, [60000] + MANY, 1, (2, 4, 8), 1 << 20, 0.1, 1, True, "later"),   # the paper's formats
    (64, 4, 8, [900, 300] * 36, 0, (8, 2, 4), 128, 0.3, 2, False, None),
    (128, 8, 8, [700, 90] * 36, 0, (4, 8, 2), 128, 0.3, 2, False, None),
    (64, 8, 8, [300, 120] * 128, 0, (8, 2, 4), 128, 0.0, 8, True, None),        # a wave a head, four without one
    (64, 4, 8, [400, 40] * 128, 0, (8, 2, 4), 60, 0.3, 8, False, None),
    (128, 5, 8, [400, 200] * 128, 0, (2, 4, 8), 60, 0.3, 8, False, None),
    (64, 8, 12, [300, 70] * 90, 0, (8, 2, 4), 60, 0.3, 8, False, None),         # the last workgroup of a sequence has four of eight heads
    (128, 4, 12, [300, 70] * 90, 1, (2, 4, 8), 60, 0.3, 8, True, None),
    (64, 4, 8, [300, 120] * 128, 1, (2, 4, 8), 60, 0.2, 8, True, None),
], ids=lambda x: str(x)[:24].replace(" ", ""))
def test_window_lists_and_groups(D, G, H, ctx, fmt, bits, window, share, hg, by_page, overflow):
    """lists of pages and of quads, longer than they can be, and several heads to a workgroup.  Against the plain kernel, and, for the statistic, against
    full attention once everything outside the window is evicted"""
    print("window, lists and groups:", D, G, H, len(ctx), max(ctx), fmt, bits, window, share, flush=True)
    c, q = _cache(D, G, H, ctx, fmt, bits, 41 + D + G)
    q_pos = _reuse(c, ctx, np.random.default_rng(D + G + len(ctx)), share) if share else [x - 1 for x in ctx]
    if window < 0:
        window = q_pos[0] + 1 - ctx[0]
    S, pages = q.shape[0], int(c.n_pages[:, 0].sum(-1).max())
    heads, waves = _grouping(c, S)
    entries, kind, first = _visible(c, 0, q_pos[0], window, waves, heads)
    print("entries", entries, "in the first block", first, "pages" if kind else "quads", flush=True)
    assert heads == hg and kind == by_page
    assert (max(entries) > LIST) == (overflow is not None) and (max(first) > LIST) == (overflow == "first")
    assert overflow != "later" or (0 < max(first) < LIST)
    (o, l), (ro, rl) = _both(c, q, D, window=window, q_pos=q_pos)
    # (five items of four waves share a head in the plain kernel, which adds token by token; a page more or less moves an output by 4 / tokens, ten times that)
    _close(o, l, ro, rl, least=1.2e-7 * max(100, min(window, max(ctx)) / 20) ** 0.5)
    ids, qp = torch.arange(S, dtype=torch.int32, device="cuda:0"), _put(q_pos)
    got = []
    for w in (window, 0):
        out, sp = torch.empty((S, G * H, D), dtype=torch.float32, device="cuda:0"), torch.empty(S, dtype=torch.float32, device="cuda:0")
        B.thinkv_decode_attention_sparsity(c, 0, q, out, None, sp, ids, qp, w, D ** -0.5, pages)
        got.append((out, sp))
        if w:
            for b in range(S):
                for k in range(3):
                    live, pos = _live(c, b, k)
                    old = np.flatnonzero((live & (pos <= q_pos[b] - window)).reshape(-1))
                    if len(old):
                        B.thinkv_evict(c, 0, _put(np.full(len(old), b)), _put(k << 28 | old))
    # (scores alike up to the order of a few additions: one entry in a thousand, or one of a short context, may change sides)
    n = torch.tensor([min(x + 1, window) for x in q_pos], device="cuda:0")
    assert float(((got[0][1] - got[1][1]).abs() - 1.0 / (n * H)).max()) <= 1e-3 and float(got[1][1].max()) > 1e-3
    assert float((got[0][0] - got[1][0]).abs().max()) <= 1e-4


@pytest.mark.parametrize("D,G,ctx,fmt,dead,bound", [
    (128, 4, [3000, 17, 1], 0, 0.6, None), (64, 8, [5000, 300], 0, 0.6, 100), (128, 2, [900], 1, 0.6, None), (64, 4, [200, 40], 0, 1.0, None)])
def test_sparsity_of_pages_with_nothing_live(D, G, ctx, fmt, dead, bound):
    """full attention counts by the masks: what the workspace held before does not matter, and a window over everything (which
    clears the scores first) gives the same"""
    print("sparsity with dead pages:", D, G, ctx, fmt, dead, bound, flush=True)
    c, q = _cache(D, G, 3, ctx, fmt, (8, 2, 4), 5 + D, dead=dead)
    S, Hq = q.shape[:2]
    ids = torch.arange(S, dtype=torch.int32, device="cuda:0")
    qp = torch.full((S,), 1 << 20, dtype=torch.int32, device="cuda:0")
    pages = int(c.n_pages[:, 0].sum(-1).max()) if bound is None else bound
    need = B.load().thinkv_decode_sparsity_workspace_bytes(B.C.byref(c.cfg), S, pages)
    got = []
    for junk, window in ((float("nan"), 0), (3e38, 0), (0.0, 1 << 21)):
        ws = torch.full((need // 4,), junk, dtype=torch.float32, device="cuda:0")
        out, sp = torch.empty((S, Hq, D), dtype=torch.float32, device="cuda:0"), torch.empty(S, dtype=torch.float32, device="cuda:0")
        rc = B.load().thinkv_decode_attention_sparsity(B.C.byref(c.view), 0, B._ptr(q), B._ptr(out), B._ptr(None), B._ptr(sp), B._ptr(ids), B._ptr(qp), S,
                                                       window, D ** -0.5, B.BF16, B.F32, pages, B._ptr(ws), need, B._stream(None))
        torch.cuda.synchronize()
        assert rc == 0
        got.append(sp.cpu())
    assert torch.equal(got[0], got[1])
    # the two attention kernels round scores alike up to the order of a few additions: one entry in a thousand may change sides
    assert float((got[0] - got[2]).abs().max()) <= 1e-3


@pytest.mark.parametrize("D,G,fmt,window", [(128, 4, 0, 0), (128, 8, 0, 0), (64, 8, 0, 0), (64, 3, 1, 0), (128, 8, 1, 0),
                                            (128, 4, 0, 200), (64, 8, 1, 200)])
def test_a_query_head_that_is_not_finite_stays_alone(D, G, fmt, window):
    """one head of a group holds a NaN, an infinity, or a bf16 number above binary16's range: the heads that share its kv-head
    get what the plain kernel gives them, and the head itself the result of a denominator that is not a number"""
    print("stream, one head not finite:", D, G, fmt, window, flush=True)
    ctx = [900, 700, 300]
    c, q = _cache(D, G, 2, ctx, fmt, (8, 2, 4), 31 + D + G, dead=0.1)
    bad = torch.zeros((len(ctx), 2 * G), dtype=torch.bool)
    for s, x in enumerate((float("nan"), float("inf"), 1e5)):
        head = (s + 1) % G
        q[s, head, 5 + s] = x
        bad[s, head] = True
    (o, l), (ro, rl) = _both(c, q, D, window=window, q_pos=[x - 1 for x in ctx])
    assert bool(torch.isfinite(ro[~bad]).all()) and bool(torch.isfinite(rl[~bad]).all())
    assert float((o - ro)[~bad].abs().max()) <= 1e-4 * max(1.0, float(ro[~bad].abs().max()))
    assert float((l - rl)[~bad].abs().max()) <= 1e-4
    assert bool((o[bad] == 0).all()) and bool((l[bad] == -float("inf")).all())


@pytest.mark.parametrize("D,G,H,ctx,fmt,ids,bound", [
    (128, 4, 8, [6500] * 17, 0, None, None),                               # 136 heads: neither one nor two to a compute unit
    (64, 8, 3, [9000, 30, 0, 1, 4000, 700] * 9, 0, None, None),            # uneven lengths, an empty sequence
    (64, 2, 1, [40] * 180 + [9000] * 4 + [4100] * 20, 1, None, None),      # more sequences than lanes of a wave
    (128, 8, 8, [6000] * 20 + [300] * 20, 1, None, None),                  # more heads than compute units
    (128, 1, 2, [20000, 100], 0, [0, 1, 0, -1, 7, 1], None),               # a sequence asked for twice, and two that do not exist
    (128, 4, 4, [9000, 2500, 800], 0, None, 300),                          # the host's bound is too low for the first
    (128, 4, 4, [2500, 800, 90], 0, None, 40000),                          # ... and far too high
], ids=lambda x: str(x)[:24].replace(" ", ""))
def test_items_dealt_over_a_batch(D, G, H, ctx, fmt, ids, bound):
    """every (query, kv-head) gets at least one item and rows of its own, the longer sequences more; results as the plain kernel's"""
    print("stream, dealt:", D, G, H, len(ctx), max(ctx), fmt, ids, bound, flush=True)
    c, q = _cache(D, G, H, ctx, fmt, (8, 2, 4), 41 + D + G + len(ctx))
    seqs = list(range(len(ctx))) if ids is None else ids   # (a call takes as many queries as the cache has sequences)
    for k in range(0, len(seqs), len(ctx)):
        part = seqs[k:k + len(ctx)]
        items = []
        (o, l), (ro, rl) = _both(c, q[:len(part)], D, bound, ids=part, items=items)
        n, row0 = items
        pages = c.n_pages[:, 0].sum(-1).cpu()
        mine = torch.tensor([int(pages[s]) if 0 <= s < len(ctx) else 0 for s in part])
        assert bool(((n >= 1) & (n <= 1024) & (row0 >= 0) & (row0 < 1 << 16)).all()) and (int(n.max()) > 1 or int(mine.max()) < 100)
        assert bool((n == n[:, :1]).all())                                  # the heads of a sequence share alike
        order = torch.argsort(mine)
        assert bool((n[order, 0].diff() >= 0).all())
        rows = torch.cat([torch.arange(int(r), int(r) + int(m)) for r, m in zip(row0.flatten(), n.flatten())])
        assert len(rows.unique()) == len(rows)
        _close(o, l, ro, rl)


@pytest.mark.parametrize("D,G,window", [(128, 4, 0), (128, 8, 0), (64, 8, 0), (64, 3, 0), (128, 4, 700)])
def test_every_code_of_the_papers_formats(D, G, window):
    """keys and values that take every E4M3 code (subnormal ones included), and groups of many sizes for the other types: each
    code reaches the matrix cores as the number that it is, in its own channel and slot"""
    print("stream, every code:", D, G, window, flush=True)
    H, n, scale = 2, 3 * 16 * 40, 0.0625
    code = np.arange(127)
    mag = np.where(code < 8, code * 2.0 ** -9, (1 + code % 8 / 8.0) * 2.0 ** (code // 8 - 7.0)) * scale
    rng = np.random.default_rng(71 + D + G)
    at = (np.arange(n * H * D) * 31 + rng.integers(0, 3, n * H * D)) % 127   # (a permutation of the codes, shaken)
    row = lambda: torch.from_numpy((mag[rng.permutation(at)] * rng.choice([-1.0, 1.0], n * H * D)).reshape(n, H, D)).to("cuda:0").float()  # noqa: E731
    c = B.Cache(1, G * H, H, D, (8, 4, 2), 1, n // 16 + 3, [n // 16 + 3] * 3, fmt=B.FMT_FP, fp8_scale=(scale, scale))
    d = lambda x: torch.from_numpy(x).to("cuda:0")  # noqa: E731
    k, v = row(), row()
    B.thinkv_append_quantized(c, 0, k, v, d(np.zeros(n, np.int32)), d(np.arange(n, dtype=np.int32)), d((np.arange(n) // 16 % 3).astype(np.uint8)),
                              torch.empty(n, dtype=torch.int32, device="cuda:0"))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(D + G)
    q = (torch.randn((1, G * H, D), generator=gen, device="cuda:0") * 0.05).to(torch.bfloat16)
    (o, l), (ro, rl) = _both(c, q, D, window=window, q_pos=[n - 1])
    _close(o, l, ro, rl)
