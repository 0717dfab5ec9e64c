"""Survivor choice at the edges of its kernels: one to four workgroups to a segment's products, or a kernel that does it all (head counts, segment sizes and
the room for the parts), rows at tile edges, segments larger than half a compute unit holds (192 points), tokens outside every
segment, both number formats.  Keys, the last Lloyd step and the survivors as in test_gpu_tbe, against the oracle's keys."""
import numpy as np
import pytest
import torch

import parity
from oracle import tbe as otbe
from paper_2510_01290_amd import synth
from test_gpu_tbe import MIN_MARGIN, _check_clustering, _gpu_select

pytestmark = pytest.mark.gpu

SIZES = [2, 15, 16, 17, 33, 64, 65, 127, 129, 191, 192, 193, 224, 225, 256]
KEEPS = [1, 8, 4, 16, 32, 63, 64, 64, 5, 64, 3, 33, 64, 64, 16]


@pytest.mark.parametrize("heads,D,fmt,bits", [(1, 64, "int", (8, 2, 4)), (3, 64, "fp", (2, 4, 8)), (9, 64, "int", (2, 4, 8)),
                                              (4, 128, "int", (8, 2, 4)), (5, 128, "fp", (2, 4, 8)), (16, 128, "int", (4, 4, 4)),
                                              (32, 128, "int", (8, 2, 4))])
def test_select_at_the_edges(heads, D, fmt, bits):
    print("survivor choice at the edges", heads, D, fmt, bits, flush=True)
    geom = synth.Geometry(1, heads, heads, D, "f16", bits, fmt)
    sizes, keeps = (SIZES, KEEPS) if heads < 32 else (SIZES[9:], KEEPS[9:])       # (the oracle takes seconds a million channels)
    wl = synth.bulk_evict_refill("tbe-edges", geom, 61, 1, np.array([sum(sizes) + 90]), {synth.E: 0.1}, refill=0)
    gc = parity.make_gpu_cache(wl)
    gr = synth.ScriptRunner(wl, parity.GpuBackend(gc)).run()
    ob = parity.make_oracle(wl)
    synth.ScriptRunner(wl, ob).run()
    dead = {(int(s), int(p)) for op in wl.ops if isinstance(op, synth.Evict) for s, p in zip(op.seqs, op.pos)}
    hs = gr.handle[(0, 0)]
    live = np.array([int(hs[p]) for p in range(int(wl.q_pos[0]) + 1) if hs[p] != -1 and (0, p) not in dead], np.int32)
    while sum(sizes) + 12 > len(live):            # the evictions took some: the last segments go
        sizes, keeps = sizes[1:], keeps[1:]
    off = (7 + np.concatenate([[0], np.cumsum(sizes)])).astype(np.int32)      # seven tokens before the first segment, five behind
    th = live[:off[-1] + 5]
    ts, keep = np.zeros(len(th), np.int32), np.array(keeps, np.int32)
    got, x, cent, assign = _gpu_select(gc, 0, ts, th, off, keep, inspect=True)
    stored = otbe.segment_keys(ob.cache, 0, 0, th)
    assert np.abs(x - stored).max() <= 1e-6 * np.abs(stored).max()            # binary32 rows of every listed token
    inner = slice(off[0], off[-1])
    n = _check_clustering(gc, ob, 0, ts, th, off, keep, 8, got, x, cent, assign)
    assert n == len(keeps)
    want, margins = otbe.select_evictions(ob.cache, 0, ts[inner], th[inner], off - off[0], keep, 8)
    clear = 0
    for sg, (a, b) in enumerate(zip(off[:-1], off[1:])):
        if margins[sg] > MIN_MARGIN:
            clear += 1
            assert np.array_equal(got[a:b], want[a - off[0]:b - off[0]]), (sg, margins[sg])
    assert clear >= len(keeps) // 2
    assert (got[:off[0]] == 12345).all() and (got[off[-1]:] == 12345).all()   # tokens of no segment: untouched
    assert int(gc.dev_status.abs().sum().item()) == 0


def test_a_key_that_is_no_number_spoils_its_own_cluster_only():
    """a token whose scales are infinite: its products are not numbers, it joins the first cluster; the others are clustered as
    they are without it, but for that cluster"""
    print("a key that is no number", flush=True)
    geom = synth.Geometry(1, 2, 2, 64, "f16", (8, 2, 4))
    wl = synth.bulk_evict_refill("tbe-nan", geom, 62, 1, np.array([200]), {}, refill=0)
    gc = parity.make_gpu_cache(wl)
    gr = synth.ScriptRunner(wl, parity.GpuBackend(gc)).run()
    hs = gr.handle[(0, 0)]
    th = np.array([int(h) for h in hs[:150]], np.int32)
    cls, pi, slot = th[70] >> 28, (th[70] >> 4) & 0xFFFFFF, th[70] & 15
    pid = int(gc.block_table[0, 0, cls, pi].item())
    block = gc.page_bytes[cls] // 2
    codes = 64 * 2 * gc.bits_of_class[cls]
    at = pid * gc.page_bytes[cls] + codes + 2 * ((slot >> 2) * 8 + (slot & 3))   # scale of group 0, head 0
    assert at < (pid + 1) * gc.page_bytes[cls] and block > codes
    gc.arena[cls][at:at + 2] = torch.tensor([0x00, 0x7C], dtype=torch.uint8, device=gc.device)
    off, keep = np.array([0, 150], np.int32), np.array([12], np.int32)
    got, x, cent, assign = _gpu_select(gc, 0, np.zeros(150, np.int32), th, off, keep, inspect=True)
    assert not np.isfinite(x[70]).all() and np.isfinite(np.delete(x, 70, 0)).all()
    assert assign[70] == 0 and 1 <= (got == -1).sum() <= 12
    for j in np.unique(assign):
        assert (got[assign == j] == -1).sum() == 1
    fine = [j for j in range(1, 12) if (assign == j).any()]
    assert len(fine) >= 6 and np.isfinite(cent[0, fine]).all()


@pytest.mark.parametrize("heads,D", [(1, 64), (2, 64), (1, 128), (7, 64), (8, 64), (9, 64), (8, 128), (32, 128)])
def test_the_smallest_workspace_is_enough(heads, D):
    """keys, centroids, clusters and 256 bytes, at an address that is no multiple of 256; what lies around it is left alone"""
    print("the smallest workspace", heads, D, flush=True)
    import ctypes as C
    from paper_2510_01290_amd import binding as B
    sizes, keeps = [256, 192, 193, 100, 30], [64, 64, 33, 16, 4]
    n, n_seg = sum(sizes), len(sizes)
    geom = synth.Geometry(1, heads, heads, D, "f16", (8, 2, 4))
    wl = synth.bulk_evict_refill("tbe-ws", geom, 66, 1, np.array([n]), {}, refill=0)
    gc = parity.make_gpu_cache(wl)
    gr = synth.ScriptRunner(wl, parity.GpuBackend(gc)).run()
    th = np.array([int(h) for h in gr.handle[(0, 0)][:n]], np.int32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    want, x, cent, assign = _gpu_select(gc, 0, np.zeros(n, np.int32), th, off, np.array(keeps, np.int32), inspect=True)
    size = 4 * (n * heads * D + n_seg * 64 * heads * D + n) + 256
    buf = torch.full((size + 1024,), 0x5A, dtype=torch.uint8, device=gc.device)
    assert buf.data_ptr() % 256 == 0
    args = [torch.from_numpy(a).to(gc.device) for a in (np.zeros(n, np.int32), th, off, np.array(keeps, np.int32))]
    ev = torch.empty(n, dtype=torch.int32, device=gc.device)
    call = lambda nb: B.load().thinkv_tbe_select(C.byref(gc.view), 0, *[a.data_ptr() for a in args], n_seg, n, 8, ev.data_ptr(), buf.data_ptr() + 16, nb, None)  # noqa: E731
    assert call(size - 1) == 4                                       # too small
    torch.cuda.synchronize()
    assert (buf == 0x5A).all()
    assert call(size) == 0
    torch.cuda.synchronize()
    assert (buf[:16] == 0x5A).all() and (buf[16 + size:] == 0x5A).all()
    assert np.array_equal(ev.cpu().numpy(), want)
    f = buf[256:256 + 4 * (n * heads * D)].view(torch.float32).view(n, -1).cpu().numpy()
    assert np.array_equal(f.astype(np.float64), x)


@pytest.mark.parametrize("heads", [3, 9])                             # one kernel that does it all, and three
@pytest.mark.parametrize("before,behind", [(0, 0), (0, 1), (3, 0), (65, 900), (1300, 2), (700, 700)])
def test_rows_of_tokens_that_are_not_clustered(before, behind, heads):
    """tokens before, behind and in segments that keep all they have or are too large: their rows are written, each once"""
    print("rows outside", before, behind, heads, flush=True)
    geom = synth.Geometry(1, heads, heads, 64, "f16", (8, 2, 4))
    sizes, keeps = [3, 64, 300, 20, 1, 7], [8, 64, 64, 9, 1, 64]
    total = before + sum(sizes) + behind
    wl = synth.bulk_evict_refill("tbe-rows", geom, 65, 1, np.array([total]), {}, refill=0)
    gc, ob = parity.make_gpu_cache(wl), parity.make_oracle(wl)
    gr = synth.ScriptRunner(wl, parity.GpuBackend(gc)).run()
    synth.ScriptRunner(wl, ob).run()
    th = np.array([int(h) for h in gr.handle[(0, 0)][:total]], np.int32)
    off = (before + np.concatenate([[0], np.cumsum(sizes)])).astype(np.int32)
    gc.workspace(1 << 23).fill_(0x7F)
    got, x, _, assign = _gpu_select(gc, 0, np.zeros(total, np.int32), th, off, np.array(keeps, np.int32), inspect=True)
    stored = otbe.segment_keys(ob.cache, 0, 0, th)
    assert np.abs(x - stored).max() <= 1e-6 * np.abs(stored).max()
    assert (got[:before] == 12345).all() and (got[off[-1]:] == 12345).all()
    clustered = np.zeros(total, bool)
    clustered[off[3]:off[4]] = True
    assert (got[before:off[-1]][~clustered[before:off[-1]]] == -1).all() and (got[clustered] == -1).sum() <= 9


@pytest.mark.parametrize("fmt,heads,D", [("int", 3, 64), ("int", 5, 128), ("fp", 9, 64), ("fp", 3, 128)])
def test_a_token_that_does_not_exist_is_the_origin(fmt, heads, D):
    """handles that name no page, inside a clustered segment whose size is no multiple of a tile and behind it: rows of zeros, flagged"""
    print("tokens that do not exist", fmt, heads, D, flush=True)
    from paper_2510_01290_amd import binding as B
    geom = synth.Geometry(1, heads, heads, D, "f16", (2, 4, 8), fmt)
    wl = synth.bulk_evict_refill("tbe-none", geom, 64, 1, np.array([120]), {}, refill=0)
    gc = parity.make_gpu_cache(wl)
    gr = synth.ScriptRunner(wl, parity.GpuBackend(gc)).run()
    th = np.array([int(h) for h in gr.handle[(0, 0)][:75]], np.int32)
    none = [0, 17, 40, 73]
    th[none] = 1 << 28 | 4000 << 4
    got, x, cent, assign = _gpu_select(gc, 0, np.zeros(75, np.int32), th, np.array([0, 70], np.int32), np.array([9], np.int32), inspect=True)
    assert (x[none] == 0).all() and (np.delete(np.abs(x).sum(1), none) > 0).all()
    assert len(set(assign[[0, 17, 40]])) == 1 and 1 <= (got[:70] == -1).sum() <= 9
    assert gc.dev_status.cpu().numpy()[0] & B.ST_BAD_SLOT


def test_a_cluster_that_gets_its_members_back():
    """Cluster 1 loses all its members in the second assignment and gets exactly them back in the third: its centroid has not moved,
    but the distances of its members to it are asked for again.  (Found by a search on the CPU: with the distances to the
    clusters that they were in meanwhile, token 9 would stay instead of token 1.)  Whole numbers, exact in the 8-bit format."""
    print("a cluster that gets its members back", flush=True)
    at = np.array([(70, 44), (66, 22), (0, 22), (60, 61), (63, 20), (60, 63), (181, 7), (2, 27), (62, 40), (123, 3),
                   (125, 40), (186, 61), (70, 60), (180, 1), (62, 60), (180, 1), (1, 19), (125, 57), (127, 61), (6, 2)])
    n, k, iters = len(at), 5, 3
    geom = synth.Geometry(1, 1, 1, 64, "f16", (8, 2, 4))
    classes = [np.full(n, synth.T, np.uint8)]
    wl = synth.Workload("tbe-back", geom, 63, 1, classes, [], (0,), np.array([n - 1], np.int32))
    pages = n // 16 + 4
    gc = parity.make_gpu_cache(wl, arena_pages=(pages,) * 3, max_pages=pages)
    ob = parity.make_oracle(wl, arena_pages=(pages,) * 3, max_pages=pages)
    gb = parity.GpuBackend(gc)
    rows = torch.zeros((n, 1, 64), dtype=torch.float16)
    for g in range(2):                            # a group's extremes are the same in every token: its scale is 1
        rows[:, 0, 32 * g + 1] = 255
        rows[:, 0, 32 * g + 5] = torch.from_numpy(at[:, g].copy()).to(torch.float16)
    th = np.asarray(gb.append(0, rows.to(gc.device), rows.to(gc.device), np.zeros(n, np.int64), np.arange(n), classes[0])).astype(np.int32)
    ob.append(0, rows, rows, np.zeros(n, np.int64), np.arange(n), classes[0])
    assert np.array_equal(otbe.segment_keys(ob.cache, 0, 0, th)[:, [5, 37]], at)
    ts, off, keep = np.zeros(n, np.int32), np.array([0, n], np.int32), np.array([k], np.int32)
    want, margins = otbe.select_evictions(ob.cache, 0, ts, th, off, keep, iters)
    assert margins[0] > MIN_MARGIN and want[1] == -1 and want[9] != -1
    got = _gpu_select(gc, 0, ts, th, off, keep, max_iters=iters)
    assert np.array_equal(got, want)
