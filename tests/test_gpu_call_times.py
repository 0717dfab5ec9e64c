"""Calls of one kind at two sizes, timed in turn in one process: a path that only one of the two takes must not be slower out of proportion to
the work.  The bounds lie about halfway (in factors) between what is measured and what the fault that each one names took."""
import numpy as np
import pytest
import torch

from paper_2510_01290_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _put(x, t=torch.int32):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV, t)


def _ratio(slow, fast, n=8):
    """median over five turns of the time of slow() over that of fast()"""
    times = []
    for f in (slow, fast):
        f()
    for _ in range(5):
        t = []
        for f in (slow, fast):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            f()
            a.record()
            for _ in range(n):
                f()
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) / n)
        times.append(t[0] / t[1])
    print("ratio", sorted(times)[2], "of", t[0] * 1000, "to", t[1] * 1000, "us", flush=True)
    return sorted(times)[2]


def _filled(S, n, hkv, D, bits=(4, 4, 4), types=1):
    """S sequences of n tokens, and the tokens' handles [S, n]"""
    c = B.Cache(1, hkv, hkv, D, bits, S, n // 16 + 8, (S * (n // 16 + 8),) * 3)
    g = torch.Generator(device=DEV)
    g.manual_seed(S + n)
    rows = torch.randn((S * n, hkv, D), generator=g, device=DEV).half()
    h = torch.empty(S * n, dtype=torch.int32, device=DEV)
    cls = np.tile(np.arange(n) // 64 % types, S)
    B.thinkv_append_quantized(c, 0, rows, rows, _put(np.repeat(np.arange(S), n)), _put(np.tile(np.arange(n), S)), _put(cls, torch.uint8), h)
    return c, h.cpu().numpy().reshape(S, n)


def test_a_plan_into_lists_that_are_too_short():
    """2,048 sequences, room for a quarter of their cuts: 46 times the call with room for all where every workgroup looked at the
    sequences before it one after the other, 1.7 times where it looks at 64 at a time"""
    S, n = 2048, 256
    c, _ = _filled(S, n, 1, 64)
    start = np.zeros((S, 4), np.int32)
    start[:] = np.arange(4) * 64
    args = (_put(np.arange(S)), _put(start), _put(np.zeros((S, 4)), torch.uint8), _put(np.full(S, 4)), _put(np.ones(S), torch.uint8), 0, 64)
    z = lambda k: torch.zeros(k, dtype=torch.int32, device=DEV)              # noqa: E731
    lists = {share: (z(S * n // share), z(S * n // share), z(S * 3 // share + 1), z(S * 3 // share), z(2)) for share in (1, 4)}
    call = lambda share: B.thinkv_tbe_plan(c, 0, *args, *lists[share], rule=B.TBE_BY_SIZE)   # noqa: E731
    r = _ratio(lambda: call(4), lambda: call(1))
    assert lists[4][4][0] == S * 3 // 4 and r < 9.0


def _select(c, handles, first, sizes, keep, n_tok):
    """thinkv_tbe_select over the first n_tok tokens of the sequences in a row, segments from token `first` on"""
    S, n = handles.shape
    off = first + np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] <= n_tok <= S * n and all(a // n == (b - 1) // n for a, b in zip(off[:-1], off[1:]))
    args = (_put(np.repeat(np.arange(S), n)[:n_tok]), _put(handles.reshape(-1)[:n_tok]), _put(off), _put(np.full(len(sizes), keep)),
            torch.empty(n_tok, dtype=torch.int32, device=DEV))
    return lambda: B.thinkv_tbe_select(c, 0, *args)


def test_tokens_outside_every_segment():
    """32 segments with 28,000 tokens behind them: 16 times the call without those where four workgroups wrote the rows of all, now 1.3"""
    c, h = _filled(32, 1024, 8, 128, (8, 2, 4), 3)
    sizes = [128] * 32
    assert _ratio(_select(c, h, 0, sizes, 32, 32 * 1024), _select(c, h, 0, sizes, 32, 4096)) < 5.0


@pytest.mark.parametrize("hkv,D,was,now,most", [(8, 128, 2.45, 1.68, 2.1), (2, 64, 2.24, 1.44, 1.8)])
def test_segments_of_more_than_192_tokens(hkv, D, was, now, most):
    """a segment of 256 tokens against one of 192 (1.8 times the pairs): `was` where the products of the points behind the 192nd were read from
    memory one after the other and the channels were walked twice"""
    c, h = _filled(1, 512, hkv, D, (8, 2, 4), 3)
    assert _ratio(_select(c, h, 0, [256], 64, 256), _select(c, h, 0, [192], 64, 192)) < most, (was, now)
