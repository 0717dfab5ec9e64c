"""The eviction plan where a sequence has more segments than a wave looks at in one go, where the budget, the limit of cuts or
the output lists end the walk in the middle, and where pages are more than a workgroup walks in one pass; against the
oracle's plan, exactly (integers)."""
import numpy as np
import pytest
import torch

import parity
from oracle import tbe as otbe
from paper_2510_01290_amd import synth
from test_gpu_tbe import _device_plan, _oracle_plan

pytestmark = pytest.mark.gpu


def _built(lens, seed):
    geom = synth.Geometry(1, 2, 2, 64, "f16", (8, 2, 4))
    rng = np.random.default_rng(seed)
    S = len(lens)
    classes = [np.repeat(rng.integers(0, 3, n // 5 + 1), 5)[:n].astype(np.uint8) for n in lens]
    wl = synth.Workload("tbe-plan-long", geom, seed, S, classes, [], (0,), np.array(lens, np.int32) - 1)
    pages = max(lens) // 16 + 8
    gc = parity.make_gpu_cache(wl, arena_pages=(S * pages,) * 3, max_pages=pages)
    ob = parity.make_oracle(wl, arena_pages=(S * pages,) * 3, max_pages=pages)
    gb = parity.GpuBackend(gc)
    for s in range(S):
        k = synth.kv_rows(seed, 0, s, 0, 0, lens[s], geom, torch.device("cpu"))
        h = gb.append(0, k.to(gc.device), k.to(gc.device), np.full(lens[s], s), np.arange(lens[s]), classes[s])
        ob.append(0, k, k, np.full(lens[s], s), np.arange(lens[s]), classes[s])
        gone = rng.choice(lens[s], size=lens[s] // 6, replace=False)
        gb.evict(0, np.full(len(gone), s), h[gone])
        ob.evict(0, np.full(len(gone), s), h[gone])
    return gc, ob, rng


def _segment_table(rng, lens, width, longest):
    st, ty, ns = np.zeros((len(lens), width), np.int32), np.zeros((len(lens), width), np.uint8), np.zeros(len(lens), np.int32)
    for s, n in enumerate(lens):
        cuts = np.cumsum(rng.integers(1, longest + 1, width))
        cuts = np.concatenate([[0], cuts[cuts < n]])[:width]
        st[s, :len(cuts)], ns[s] = cuts, len(cuts)
        ty[s, :len(cuts)] = rng.integers(0, 3, len(cuts))
    return st, ty, ns


@pytest.mark.parametrize("longest,trans,budget,max_cuts,cap_seg,cap_tok", [
    (14, None, 700, 256, 2048, 1 << 16),          # the budget ends the walk, some hundred segments a type
    (14, None, 0, 100, 2048, 1 << 16),            # the limit of cuts does
    (14, [1, 0, 1], 0, 256, 2048, 1 << 16),       # both cases together
    (14, [1, 1, 1], 10 ** 6, 256, 300, 1 << 16),  # the lists end in the second sequence (segments) ...
    (14, [1, 1, 1], 10 ** 6, 256, 2048, 2500),    # ... and (tokens)
    (1, None, 0, 256, 2048, 1 << 16),             # a token a segment: nothing can go
    (120, [0, 1, 0], 900, 64, 2048, 1 << 16)])    # segments of many pages
def test_tbe_plan_over_many_segments(longest, trans, budget, max_cuts, cap_seg, cap_tok):
    print("plan over many segments", longest, trans, budget, max_cuts, cap_seg, cap_tok, flush=True)
    lens = [3700, 2100, 9000]
    gc, ob, rng = _built(lens, 51)
    st, ty, ns = _segment_table(rng, lens, 1400, longest)
    dev, ora = np.zeros(st.shape, np.int32), np.zeros(st.shape, np.int32)
    for again in range(2):                        # the second call finds the counts of the first
        got = _device_plan(gc, 0, [0, 1, 2], st, ty, ns, trans, budget, max_cuts, cap_seg, cap_tok, seg_count=dev)
        w_seq, w_h, w_off, w_keep = _oracle_plan(ob.cache, 0, [0, 1, 2], st, ty, ns, trans, budget, max_cuts, cap_seg, cap_tok, seg_count=ora)
        n_seg, n_tok = got["counts"].tolist()
        assert (n_seg, n_tok) == (len(w_keep), len(w_h)), again
        assert np.array_equal(got["seg_keep"][:n_seg], w_keep) and np.array_equal(got["seg_offset"][:n_seg + 1], w_off)
        assert np.array_equal(got["tok_handle"][:n_tok], w_h) and np.array_equal(got["tok_seq"][:n_tok], w_seq)
        assert np.array_equal(dev, ora)
    assert int(gc.dev_status.abs().sum().item()) == 0


@pytest.mark.parametrize("share_seg,share_tok,max_cuts", [(1.0, 0.9, 256), (0.35, 1.0, 256), (1.0, 0.3, 256), (0.7, 0.02, 256), (0.01, 1.0, 256), (0.5, 0.5, 3), (0.0, 1.0, 8)])
def test_tbe_plan_of_many_sequences_into_short_lists(share_seg, share_tok, max_cuts):
    """sequences by the hundred: some fit whole, some in part, some only because an earlier one was passed over; the lists end anywhere"""
    print("plan into short lists", share_seg, share_tok, max_cuts, flush=True)
    rng = np.random.default_rng(52)
    lens = rng.integers(30, 260, 150).tolist()
    gc, ob, rng = _built(lens, 53)
    st, ty, ns = _segment_table(rng, lens, 20, 60)
    order = rng.permutation(150).tolist()
    trans = (rng.random(150) < 0.8).astype(np.uint8).tolist()
    full = _oracle_plan(ob.cache, 0, order, st, ty, ns, trans, 60, max_cuts, 1 << 14, 1 << 16, rule=otbe.BY_SIZE)
    cap_seg, cap_tok = max(1, int(share_seg * len(full[3]))), max(1, int(share_tok * len(full[1])))
    dev, ora = np.zeros(st.shape, np.int32), np.zeros(st.shape, np.int32)
    for again in range(2):
        got = _device_plan(gc, 0, order, st, ty, ns, trans, 60, max_cuts, cap_seg, cap_tok, seg_count=dev)
        w_seq, w_h, w_off, w_keep = _oracle_plan(ob.cache, 0, order, st, ty, ns, trans, 60, max_cuts, cap_seg, cap_tok, seg_count=ora)
        n_seg, n_tok = got["counts"].tolist()
        assert (n_seg, n_tok) == (len(w_keep), len(w_h)), again
        assert np.array_equal(got["seg_keep"][:n_seg], w_keep) and np.array_equal(got["seg_offset"][:n_seg + 1], w_off)
        assert np.array_equal(got["tok_handle"][:n_tok], w_h) and np.array_equal(got["tok_seq"][:n_tok], w_seq)
        assert np.array_equal(dev, ora)


@pytest.mark.parametrize("max_cuts", [1, 16, 17, 64, 65])
def test_tbe_plan_sorts_lists_of_long_segments(max_cuts):
    """lists of up to 250 tokens, sorted by the workgroup of their sequence (a wave has one, or one or two pairs of them) or, from 65 cuts on, by a launch of its own"""
    test_tbe_plan_over_many_segments(250, None, 0, max_cuts, 2048, 1 << 16)
    test_tbe_plan_over_many_segments(250, [1, 0, 1], 0, max_cuts, 60, 1 << 16)


@pytest.mark.parametrize("num,den", [(40, 1), (9, 1), (1, 2)])
@pytest.mark.parametrize("max_cuts", [20, 256])
def test_tbe_plan_of_spread_and_of_equal_positions(num, den, max_cuts):
    """lists whose positions are further apart than the row of bits reaches, close to that, or (two tokens to a position: in either order) not all different"""
    _lists_of(np.arange(1840) * num // den, 8, max_cuts)


@pytest.mark.parametrize("odd,even", [(40, 1), (1, 40), (0.5, 9), (9, 0.5), (9, 9)])
@pytest.mark.parametrize("cuts", [17, 23, 32, 33, 48])
def test_tbe_plan_of_lists_sorted_in_pairs(odd, even, cuts):
    """more cuts than waves, which take two lists at once: either of the two further apart than the row reaches, or with two tokens to a position"""
    step = np.repeat(np.where(np.arange(cuts + 1) // 16 % 2 == 1, odd, even), 230)
    _lists_of(np.concatenate([[0], np.cumsum(step)[:-1]]).astype(np.int64), cuts + 1, 64)


def _lists_of(pos, width, max_cuts):
    from paper_2510_01290_amd import binding as B
    n = len(pos)
    c = B.Cache(1, 2, 1, 64, (8, 2, 4), 1, n // 16 + 4, [n // 16 + 8] * 3)
    rng = np.random.default_rng(7)
    kv = torch.randn((n, 1, 64), device="cuda:0").half()
    ten = lambda x, t: torch.tensor(np.ascontiguousarray(x), dtype=t, device="cuda:0")
    h = torch.empty(n, dtype=torch.int32, device="cuda:0")
    B.thinkv_append_quantized(c, 0, kv, kv, torch.zeros(n, dtype=torch.int32, device="cuda:0"), ten(pos, torch.int32), ten(rng.integers(0, 3, n), torch.uint8), h)
    of = {int(a): int(p) for a, p in zip(h.cpu(), pos)}
    assert len(of) == n
    start = np.zeros((1, width), np.int32)
    start[0] = pos[np.arange(width) * 230]
    got = _device_plan(c, 0, [0], start, np.zeros((1, width), np.uint8), np.array([width], np.int32), [1], 10 ** 6, max_cuts, 64, 1 << 14, seg_count=np.zeros((1, width), np.int32))
    n_seg, n_tok = got["counts"].tolist()
    assert n_seg == width - 1 and n_tok == 230 * (width - 1)
    for i in range(n_seg):
        lo, hi = got["seg_offset"][i:i + 2]
        listed = [of[int(x)] for x in got["tok_handle"][lo:hi]]
        assert listed == sorted(pos[(pos >= start[0, i]) & (pos < start[0, i + 1])].tolist())
        assert len(set(got["tok_handle"][lo:hi].tolist())) == hi - lo
    assert not np.any(got["tok_seq"][:n_tok])
