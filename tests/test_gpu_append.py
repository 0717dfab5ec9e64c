"""Appends at the edges of their plan and of the bulk place kernel: calls around the size from which they are placed in bulk, one
to five thousand tokens a sequence (one and several ranking windows), page lists longer than the masks a thread keeps, reclaimable
slots taken across windows, new pages that stay partly empty, groups whose zero-point or scale leaves binary16's range.
Tables and bytes equal the oracle's."""
import numpy as np
import pytest
import torch

import parity
from paper_2510_01290_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,dtype,fmt,calls,classes", [
    (64, torch.bfloat16, "int", [[1, 63], [0, 65]], 3),                    # 64 tokens: small; 65: bulk
    (128, torch.float16, "int", [[256, 257, 1], [4096, 15, 4097]], 3),     # a window and one token more
    (128, torch.bfloat16, "fp", [[33, 200], [170, 16]], 3),
    (64, torch.float32, "fp", [[90, 31], [16, 64]], 2),
    (64, torch.bfloat16, "int", [[17000, 5], [6000, 700]], 1),             # lists of more than 1,024 pages
])
def test_bulk_plan_and_new_pages(D, dtype, fmt, calls, classes):
    print(f"[gpu] append D={D} {dtype} {fmt} {calls}", flush=True)
    H = 1 if calls[0][0] > 4096 else 3
    S = len(calls[0])
    rng = np.random.default_rng(D + S + classes)
    geom = synth.Geometry(1, 2 * H, H, D, "f16", (8, 4, 2), fmt=fmt) if fmt == "fp" else synth.Geometry(1, 2 * H, H, D, "f16", (8, 4, 2))
    cls = [[rng.integers(0, classes, n).astype(np.uint8) for n in call] for call in calls]
    wl = synth.Workload("append-edges", geom, 0, S, [np.concatenate([c[s] for c in cls]) for s in range(S)], [])
    gc, ob = parity.make_gpu_cache(wl), parity.make_oracle(wl)
    gb = parity.GpuBackend(gc)
    base = np.zeros(S, np.int32)
    for ci, call in enumerate(calls):
        n = sum(call)
        ts = np.repeat(np.arange(S, dtype=np.int32), call)
        tp = np.concatenate([base[s] + np.arange(call[s]) for s in range(S)]).astype(np.int32)
        gen = torch.Generator().manual_seed(ci)
        k, v = [(torch.randn((n, H, D), generator=gen) * 3).to(dtype) for _ in range(2)]
        hg = gb.append(0, k.cuda(), v.cuda(), ts, tp, np.concatenate(cls[ci]))
        ho = ob.append(0, k, v, ts, tp, np.concatenate(cls[ci]))
        assert np.array_equal(hg, ho), ci
        parity.compare_bookkeeping_full(ob.cache, gc)
        base += np.asarray(call, np.int32)
        pick = rng.random(n) < 0.4
        gb.evict(0, ts[pick], hg[pick])
        ob.evict(0, ts[pick], ho[pick])
    parity.compare_bookkeeping_full(ob.cache, gc)
    parity.compare_sequences(ob.cache, gc, [(s, s, 0) for s in range(S)], check_bytes=True)



@pytest.mark.parametrize("D,dtype,fmt,calls,classes", [
    (64, torch.bfloat16, "int", [[257], [255], [257], [513]], 3),               # one sequence: a token more than 256, where the plan takes 512 threads, and fewer
    (128, torch.bfloat16, "int", [[511, 512, 513], [1, 1600, 2]], 3),           # a token a thread, one more, and sequences with hardly any beside long ones
    (64, torch.float16, "int", [[33500], [9000]], 1),                           # lists of more pages than 512 threads keep the masks of
    (64, torch.bfloat16, "fp", [[4096, 4097], [4608, 300]], 2),                 # windows
])
def test_plan_of_long_prompts(D, dtype, fmt, calls, classes):
    test_bulk_plan_and_new_pages(D, dtype, fmt, calls, classes)


@pytest.mark.parametrize("H,D,fmt,n,heads_per_block", [(3, 64, "int", 22000, 2), (3, 64, "int", 43760, 3), (5, 64, "int", 26300, 4), (5, 128, "fp", 26300, 4),
                                                       (6, 64, "int", 22000, 4), (9, 64, "fp", 14600, 4), (8, 64, "int", 16400, 4)])
def test_heads_of_a_block(H, D, fmt, n, heads_per_block):
    """blocks of two, three and four heads, and a last one of one or two: every head's bytes are those of a cache with that head alone (whose
    tables, and whose bytes at these sizes, the tests above compare with the oracle's)"""
    from paper_2510_01290_amd import binding as B
    print(f"[gpu] append, heads of a block: H={H} D={D} {fmt} {n}", flush=True)
    per = (H * ((n + 15) // 16) + 4095) // 4096
    assert min(4 if per > 2 else per, H) == heads_per_block
    rng = np.random.default_rng(H + D)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")  # noqa: E731
    cls = np.repeat(np.arange(n), rng.integers(1, 120, n))[:n] % 3
    gen = torch.Generator(device="cuda:0").manual_seed(H)
    k, v = (torch.randn((n, H, D), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    tok = [d(x) for x in (np.arange(n, dtype=np.int32) // (n // 2 + 1), np.arange(n, dtype=np.int32), cls.astype(np.uint8))]

    def filled(heads):
        c = B.Cache(1, heads.stop - heads.start, heads.stop - heads.start, D, (8, 4, 2), 2, n // 16 + 4, [n // 16 + 8] * 3, fmt=B.FMT_FP if fmt == "fp" else B.FMT_INT,
                    fp8_scale=(0.05, 0.05))
        h = torch.empty(n, dtype=torch.int32, device="cuda:0")
        B.thinkv_append_quantized(c, 0, k[:, heads].contiguous(), v[:, heads].contiguous(), *tok, h)
        return c, h

    c, h = filled(slice(0, H))
    assert int(c.dev_status.abs().sum()) == 0 and int(c.n_live.sum()) == n
    for x in range(H):
        one, h1 = filled(slice(x, x + 1))
        assert torch.equal(h, h1) and torch.equal(c.block_table, one.block_table)
        for t in range(3):
            size = one.page_bytes[t]
            assert torch.equal(c.arena[t].view(-1, H, size)[:, x], one.arena[t].view(-1, size)), (x, t)


@pytest.mark.parametrize("n_tok", [40, 100])
def test_groups_out_of_binary16_range(n_tok):
    """zero-points that overflow to -inf and +inf next to a finite scale, ranges whose scale overflows, equal values, tiny ranges: both
    kernels give what the division gives"""
    print(f"[gpu] groups out of range, {n_tok} tokens", flush=True)
    geom = synth.Geometry(1, 2, 1, 64, "f16", (8, 4, 2))
    cls = (np.arange(n_tok) % 3).astype(np.uint8)
    wl = synth.Workload("append-range", geom, 0, 1, [cls], [])
    gc, ob = parity.make_gpu_cache(wl), parity.make_oracle(wl)
    rng = np.random.default_rng(5)
    lo = np.array([-7e4, 7e4, -3e38, 2.5, -1e-7, 0.0, -65504.0, 1e-40, 65519.0, -65520.0], np.float32)
    span = np.array([100.0, 90.0, 6e37, 0.0, 2e-7, 1e-39, 131008.0, 1e-41, 1.0, 3.0], np.float32)
    pick = rng.integers(0, len(lo), (2, n_tok, 1, 2, 1))
    x = (lo[pick] + span[pick] * rng.random((2, n_tok, 1, 2, 32), dtype=np.float32)).astype(np.float32).reshape(2, n_tok, 1, 64)
    k, v = torch.from_numpy(x[0].copy()), torch.from_numpy(x[1].copy())
    ts, tp = np.zeros(n_tok, np.int32), np.arange(n_tok, dtype=np.int32)
    hg = parity.GpuBackend(gc).append(0, k.cuda(), v.cuda(), ts, tp, cls)
    assert np.array_equal(hg, ob.append(0, k, v, ts, tp, cls))
    parity.compare_bookkeeping_full(ob.cache, gc)
    parity.compare_sequences(ob.cache, gc, [(0, 0, 0)], check_bytes=True)


@pytest.mark.parametrize("D,dtype,fmt,S,lens,share", [
    (64, torch.bfloat16, "int", 2, [9000, 300], 0.004),      # a type whose sixteen tokens lie thousands apart, over several windows
    (128, torch.float16, "fp", 3, [5000, 17, 4097], 0.02),   # ... around the distance up to which a page is written whole
    (64, torch.float32, "int", 700, [1] * 699 + [5], 0.3),   # new pages with a token or two, of more sequences than a round of sums
    (64, torch.bfloat16, "int", 90, [3, 4, 5] * 30, 0.0),    # ... around the number from which a page is written whole
], ids=lambda x: str(x)[:20].replace(" ", ""))
def test_new_pages_of_scattered_and_few_tokens(D, dtype, fmt, S, lens, share):
    print(f"[gpu] append, scattered: D={D} {dtype} {fmt} S={S} {max(lens)} {share}", flush=True)
    H = 2
    rng = np.random.default_rng(D + S)
    geom = synth.Geometry(1, 2 * H, H, D, "f16", (8, 4, 2), fmt=fmt) if fmt == "fp" else synth.Geometry(1, 2 * H, H, D, "f16", (8, 4, 2))

    def types(n):   # mostly type 2, a share of type 0, type 1 in runs
        t = np.where(rng.random(n) < share, 0, 2).astype(np.uint8)
        t[n // 3:n // 3 + n // 7] = 1
        return t

    cls = [types(n) for n in lens]
    wl = synth.Workload("append-scattered", geom, 0, S, cls, [])
    gc, ob = parity.make_gpu_cache(wl), parity.make_oracle(wl)
    gb = parity.GpuBackend(gc)
    ts = np.repeat(np.arange(S, dtype=np.int32), lens)
    tp = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    tc = np.concatenate(cls)
    gen = torch.Generator().manual_seed(S)
    k, v = (torch.randn((len(ts), H, D), generator=gen).to(dtype) for _ in range(2))
    hg = gb.append(0, k.cuda(), v.cuda(), ts, tp, tc)
    assert np.array_equal(hg, ob.append(0, k, v, ts, tp, tc))
    parity.compare_bookkeeping_full(ob.cache, gc)
    parity.compare_sequences(ob.cache, gc, [(s, s, 0) for s in range(S)], check_bytes=True)


@pytest.mark.parametrize("pages", [(1, 2, 3), (257, 1030, 4099), (5000, 9001, 0)])
@pytest.mark.parametrize("D,H", [(64, 1), (128, 8)])
def test_reset_clears_the_arenas_and_nothing_else(pages, D, H):
    """stores in fours and the rest one by one: every byte of the pages of the view, none behind them"""
    from paper_2510_01290_amd import binding as B
    c = B.Cache(1, 2 * H, H, D, (8, 2, 4), 3, 40, [n + 1 for n in pages])
    for t in c.arena + c.slot_pos:
        t.fill_(0x5A)
    for k, n in enumerate(pages):
        c.view.arena_pages[k] = n
    B.thinkv_init_view(c)
    torch.cuda.synchronize()
    for k, n in enumerate(pages):
        used = n * c.page_bytes[k]
        assert not bool(c.arena[k][:used].any()) and bool((c.arena[k][used:] == 0x5A).all())
        assert bool((c.slot_pos[k][:n] == -1).all()) and bool((c.slot_pos[k][n:] == 0x5A).all())
        assert int(c.free_top[k]) == n
