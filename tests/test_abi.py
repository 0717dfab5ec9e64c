"""The C-ABI library loads, exports every symbol the header declares, and its host-side
entry points behave without a GPU (no compute calls here)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2510_01290_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.load()


def test_every_declared_symbol_is_exported(lib):
    from paper_2510_01290_amd import binding
    hdr = open(os.path.join(ROOT, "include", "thinkv.h")).read()
    declared = set(re.findall(r"\b(thinkv_[a-z_]+)\s*\(", hdr))
    declared -= {"thinkv_status"}           # typedef names never followed by '(' anyway
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_layout_queries_match_the_stated_formula(lib):
    from paper_2510_01290_amd import binding as B
    for D in (64, 128):
        cfg = B.make_config(1, 8, 2, D, (8, 2, 4), 4, 16)
        for bits in (2, 4, 8):
            assert B.thinkv_block_bytes(cfg, bits) == 16 * 2 * (D * bits // 8 + (D // 32) * 4)
            assert B.thinkv_page_bytes(cfg, bits) == 2 * B.thinkv_block_bytes(cfg, bits)
        assert B.thinkv_block_bytes(cfg, 3) == 0
    bad = B.make_config(1, 8, 2, 96, (8, 2, 4), 4, 16)
    assert B.thinkv_block_bytes(bad, 4) == 0
    assert B.thinkv_append_workspace_bytes(cfg, 100) > 0
    assert B.thinkv_decode_workspace_bytes(cfg, 3, 100) >= 3 * 8 * (128 + 2) * 4


@pytest.mark.parametrize("heads,D", [(1, 64), (2, 64), (2, 128), (7, 64), (4, 128), (8, 128), (16, 128), (32, 128)])
def test_survivor_choice_asks_for_what_it_leaves_in_the_workspace(lib, heads, D):
    """keys, centroids and clusters, and nothing for the kernels' own use: programs hold workspaces of that size"""
    from paper_2510_01290_amd import binding as B
    cfg = B.make_config(1, heads, heads, D, (8, 2, 4), 4, 16)
    for n_tok, n_seg in [(1, 1), (700, 3), (40000, 400)]:
        assert lib.thinkv_tbe_workspace_bytes(C.byref(cfg), n_tok, n_seg) == 4 * (n_tok * heads * D + n_seg * 64 * heads * D + n_tok) + 256


@pytest.mark.parametrize("raw", [True, False])
def test_the_current_stream_with_and_without_torchs_raw_query(monkeypatch, raw):
    import importlib.util
    import types
    import torch
    from paper_2510_01290_amd import binding
    name = "_cuda_getCurrentRawStream"
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    if raw:
        monkeypatch.setattr(torch._C, name, lambda device: 0x5678 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, name, raising=False)
    spec = importlib.util.spec_from_file_location("binding_under_test", binding.__file__)
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    assert b._stream(None) == (0x567B if raw else 0x1234)
    assert b._stream(types.SimpleNamespace(cuda_stream=77)) == 77


def test_host_side_argument_errors(lib):
    from paper_2510_01290_amd import binding as B
    assert lib.thinkv_init_view(None, None) == 1
    v = B.View()
    v.cfg = B.make_config(1, 8, 2, 128, (8, 2, 4), 4, 16)
    assert lib.thinkv_init_view(C.byref(v), None) == 1            # null device pointers
    v.cfg = B.make_config(1, 8, 3, 128, (8, 2, 4), 4, 16)
    assert lib.thinkv_init_view(C.byref(v), None) == 2            # 8 heads do not group over 3
    v.cfg = B.make_config(1, 8, 2, 128, (8, 3, 4), 4, 16)
    assert lib.thinkv_evict(C.byref(v), 0, None, None, 0, None) == 2
    assert lib.thinkv_status_string(4) == b"workspace too small"
