"""thinkv_evict_append against thinkv_evict followed by thinkv_append_quantized on a second cache: lists of evictions around what a
thread holds before it applies the first (512 a workgroup), with duplicates, dead slots, placeholders and bad handles among them."""
import numpy as np
import pytest
import torch

from paper_2510_01290_amd import binding as B

pytestmark = pytest.mark.gpu


def _tables(c):
    return [c.slot_mask, c.block_table, c.n_pages, c.n_live, c.free_top, c.dev_status, *c.page_filled, *c.slot_pos, *c.page_pos_max, *c.arena]


@pytest.mark.parametrize("D,n_ev,n_new", [(64, 1, 1), (64, 255, 3), (128, 257, 64), (64, 511, 65), (64, 512, 2), (64, 513, 200), (128, 1500, 40)])
def test_evict_append_is_evict_then_append(D, n_ev, n_new):
    print("evict_append", D, n_ev, n_new, flush=True)
    dev, S, n = torch.device("cuda:0"), 3, 2400
    rng = np.random.default_rng(71 + n_ev)
    put = lambda x, t: torch.from_numpy(np.ascontiguousarray(x)).to(dev, t)      # noqa: E731
    g = torch.Generator(device=dev)
    g.manual_seed(n_ev)
    rows = lambda m: torch.randn((m, 2, D), generator=g, device=dev).half()      # noqa: E731
    seq = np.sort(rng.integers(0, S, n))
    pos = np.concatenate([np.arange((seq == s).sum()) for s in range(S)])
    k0, v0, k1, v1 = rows(n), rows(n), rows(n_new), rows(n_new)
    cls = rng.integers(0, 3, n)
    caches, handles = [], []
    for _ in range(2):
        c = B.Cache(1, 4, 2, D, (8, 2, 4), S, 120, (200, 200, 200))
        h = torch.empty(n, dtype=torch.int32, device=dev)
        B.thinkv_append_quantized(c, 0, k0, v0, put(seq, torch.int32), put(pos, torch.int32), put(cls, torch.uint8), h)
        caches.append(c)
        handles.append(h.cpu().numpy())
    assert np.array_equal(*handles)
    at = rng.integers(0, n, n_ev)                                                # with duplicates
    ev_seq, ev_h = seq[at].astype(np.int32), handles[0][at].copy()
    if n_ev > 10:
        ev_h[3], ev_seq[5], ev_h[7] = -1, S + 4, 1 << 28 | 100 << 4              # a placeholder, no such sequence, no such page
    new_seq = np.sort(rng.integers(0, S, n_new))
    args = (k1, v1, put(new_seq, torch.int32), put(n + np.arange(n_new), torch.int32), put(rng.integers(0, 3, n_new), torch.uint8))
    out = [torch.empty(n_new, dtype=torch.int32, device=dev) for _ in range(2)]
    B.thinkv_evict_append(caches[0], 0, put(ev_seq, torch.int32), put(ev_h, torch.int32), *args, out[0])
    B.thinkv_evict(caches[1], 0, put(ev_seq, torch.int32), put(ev_h, torch.int32))
    B.thinkv_append_quantized(caches[1], 0, *args, out[1])
    assert torch.equal(*out)
    for i, (a, b) in enumerate(zip(_tables(caches[0]), _tables(caches[1]))):
        assert torch.equal(a, b), i
