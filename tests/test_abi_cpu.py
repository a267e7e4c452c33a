"""Host-side checks of the C ABI: the library loads, exports every function
include/resa.h declares, computes Eq. 5 like the oracle, and rejects bad
arguments before touching the device (no call here reaches a kernel)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import oracle as O
from paper_2506_04108_amd import _lib as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    with open(os.path.join(ROOT, "include", "resa.h")) as fh:
        text = fh.read()
    return sorted(set(re.findall(r"\b(resa_[a-z0-9_]+)\s*\(", text)))


def test_exports_every_declared_symbol():
    lib = L.lib()
    names = header_functions()
    assert len(names) >= 13
    for n in names:
        assert hasattr(lib, n), f"libresa.so does not export {n}"
    assert set(names) == set(L.SIGNATURES), "binding signatures out of sync with resa.h"


def test_version():
    assert re.fullmatch(r"\d+\.\d+\.\d+", L.lib().resa_version().decode())


@pytest.mark.parametrize("s", [0.0, 0.5, 0.8, 0.9, 0.95, 0.98, 0.999999, 1.0])
def test_num_selected_matches_oracle(s):
    lib = L.lib()
    Ms = list(range(0, 5000)) + list(range(5000, 1 << 20, 997)) + [1 << 20]
    for nmin, nloc in ((0, 1), (64, 1), (256, 2), (0, 0)):
        got = [lib.resa_num_selected(M, s, nmin, nloc) for M in Ms]
        want = [O.num_selected(M, s, nmin, nloc) for M in Ms]
        assert got == want


def test_num_selected_rejects_bad_args():
    lib = L.lib()
    assert lib.resa_num_selected(-1, 0.9, 0, 1) == -1
    assert lib.resa_num_selected(10, 1.5, 0, 1) == -1
    assert lib.resa_num_selected(10, -0.1, 0, 1) == -1
    assert lib.resa_num_selected(10, 0.9, -1, 1) == -1
    assert b"invalid" in lib.resa_last_error()


FAKE = 0x100000  # 16-byte aligned stand-in address: only used on rejected calls


def cache(**kw):
    d = dict(k=FAKE, v=FAKE, kmin=FAKE, kmax=FAKE, batch=2, num_kv_heads=2, head_dim=128,
             capacity=1024, block_size=16)
    d.update(kw)
    return L.KVCacheDesc(**d)


def expect(rc, code, text):
    assert rc == code, (rc, L.lib().resa_last_error())
    assert text in L.lib().resa_last_error().decode()


def test_paged_cache_validation():
    """Paged layout: the block table must be 4-byte aligned, the pool must
    hold at least one page, and its rows must stay below 2^31."""
    lib = L.lib()
    run = lambda **kw: lib.resa_block_summarize(C.byref(cache(**kw)), FAKE, 0, -1, None)
    expect(run(block_table=FAKE + 2, num_pages=8), 1, "block_table")
    expect(run(block_table=FAKE, num_pages=0), 1, "num_pages")
    expect(run(block_table=FAKE, num_pages=1 << 26, num_kv_heads=2), 2, "2^31")


def test_summarize_validation():
    lib = L.lib()
    expect(lib.resa_block_summarize(None, FAKE, 0, -1, None), 1, "cache descriptor")
    expect(lib.resa_block_summarize(C.byref(cache(k=None)), FAKE, 0, -1, None), 1, "c->k is NULL")
    expect(lib.resa_block_summarize(C.byref(cache(v=FAKE + 8)), FAKE, 0, -1, None), 1, "aligned")
    expect(lib.resa_block_summarize(C.byref(cache(head_dim=64)), FAKE, 0, -1, None), 2, "head_dim")
    expect(lib.resa_block_summarize(C.byref(cache(block_size=8)), FAKE, 0, -1, None), 2, "block_size")
    expect(lib.resa_block_summarize(C.byref(cache(capacity=1000)), FAKE, 0, -1, None), 1, "multiple")
    expect(lib.resa_block_summarize(C.byref(cache(batch=0)), FAKE, 0, -1, None), 1, "batch")
    expect(lib.resa_block_summarize(C.byref(cache()), None, 0, -1, None), 1, "seq_lens")
    expect(lib.resa_block_summarize(C.byref(cache()), FAKE, -1, -1, None), 1, "blk_begin")
    expect(lib.resa_block_summarize(C.byref(cache()), FAKE, 5, 3, None), 1, "blk_end")
    expect(lib.resa_block_summarize(C.byref(cache()), FAKE, 0, 65, None), 1, "blk_end")


def test_append_validation():
    lib = L.lib()
    expect(lib.resa_append_kv(C.byref(cache()), FAKE, FAKE, FAKE, 1024, None), 4, "cache full")
    expect(lib.resa_append_kv(C.byref(cache()), None, FAKE, FAKE, 10, None), 1, "k_new")
    expect(lib.resa_append_kv(C.byref(cache()), FAKE, FAKE, FAKE, -1, None), 1, "max_seq_len")


def select(**kw):
    a = dict(c=C.byref(cache()), q=FAKE, hq=8, seq=FAKE, mx=1000,
             p=C.byref(L.SelectParams(0.9, 4, 1)), idx=FAKE, ns=FAKE, n_cap=64, sc=None,
             ws=FAKE, wsb=1 << 20, st=None)
    a.update(kw)
    return L.lib().resa_select_blocks(*a.values())


def test_select_validation():
    expect(select(hq=7), 1, "num_q_heads")
    expect(select(hq=18), 2, "group size")
    expect(select(q=FAKE + 4), 1, "q is not 16-byte")
    expect(select(p=None), 1, "params")
    expect(select(p=C.byref(L.SelectParams(1.2, 4, 1))), 1, "sparsity")
    expect(select(p=C.byref(L.SelectParams(0.9, -1, 1))), 1, "min_blocks")
    expect(select(mx=2000), 1, "max_seq_len")
    expect(select(n_cap=3), 4, "n_cap")
    expect(select(ws=None), 3, "workspace")
    expect(select(wsb=100), 3, "workspace")


def append_select(**kw):
    a = dict(c=C.byref(cache()), k=FAKE, v=FAKE, q=FAKE, hq=8, seq=FAKE, mx=1000,
             p=C.byref(L.SelectParams(0.9, 4, 1)), idx=FAKE, ns=FAKE, n_cap=64, sc=None,
             ws=FAKE, wsb=1 << 20, st=None)
    a.update(kw)
    return L.lib().resa_append_select(*a.values())


def test_append_select_validation():
    expect(append_select(k=None), 1, "k_new")
    expect(append_select(v=FAKE + 2), 1, "v_new")
    expect(append_select(mx=1024), 4, "cache full")
    expect(append_select(mx=-1), 1, "max_seq_len")
    expect(append_select(hq=7), 1, "num_q_heads")
    expect(append_select(n_cap=3), 4, "n_cap")
    expect(append_select(wsb=100), 3, "workspace")
    # n_cap and the workspace are sized for one token more than max_seq_len.
    lib = L.lib()
    n = lib.resa_num_selected(64, 0.9, 4, 1)
    expect(append_select(mx=1008, n_cap=lib.resa_num_selected(63, 0.9, 4, 1) - 1), 4, "n_cap")
    assert n >= 4
    need = lib.resa_select_workspace_size(2, 2, 1009, 16)
    expect(append_select(mx=1008, wsb=need - 1), 3, "workspace")


def decode(**kw):
    a = dict(c=C.byref(cache()), q=FAKE, hq=8, seq=FAKE, idx=FAKE, ns=FAKE, n_cap=16, S=0,
             sc=0.088, out=FAKE, lse=None, ws=FAKE, wsb=16, st=None)
    a.update(kw)
    return L.lib().resa_sparse_decode(*a.values())


def test_decode_validation():
    expect(decode(out=None), 1, "out")
    expect(decode(n_cap=-1), 1, "n_cap")
    expect(decode(S=-2), 1, "num_splits")
    expect(decode(sc=float("inf")), 1, "sm_scale")
    expect(decode(), 3, "decode workspace")
    need = L.lib().resa_decode_workspace_size(2, 2, 8, 16, 16, 0)
    assert need > 0
    expect(decode(ws=FAKE + 4, wsb=need), 1, "aligned")


def rectify(**kw):
    a = dict(c=C.byref(cache()), q=FAKE, k=FAKE, v=FAKE, hq=8, f=16, seq=FAKE, mask=None, mx=1000,
             sc=0.088, out=FAKE, lse=None, ref=1, ws=FAKE, wsb=16, st=None)
    a.update(kw)
    return L.lib().resa_dense_rectify(*a.values())


def test_rectify_validation():
    expect(rectify(f=0), 1, "f 0")
    expect(rectify(f=65537), 1, "f 65537")
    expect(rectify(mx=8), 1, "max_seq_len")
    expect(rectify(mx=4096), 1, "max_seq_len")
    expect(rectify(k=None), 1, "k_f")
    expect(rectify(mask=FAKE + 2), 1, "seq_mask")
    expect(rectify(), 3, "rectify workspace")
    expect(rectify(mask=FAKE), 3, "rectify workspace")


def test_workspace_sizes():
    lib = L.lib()
    full = lib.resa_select_workspace_size(8, 8, 65536, 16)
    assert full >= 8 * 8 * (4096 + 256 + 1) * 4     # scores, digit counts, tickets
    s = lib.resa_decode_num_splits(8, 8, 410, 16)
    assert 1 <= s <= 256
    assert lib.resa_decode_workspace_size(8, 8, 32, 410, 16, s) >= 64 * s * 4 * 128 * 4
    assert lib.resa_rectify_workspace_size(8, 8, 32, 32, 65664) >= 64 * 128 * 128 * 4
    # A whole-prompt window fills the chip with query blocks alone: one key split,
    # written straight to the output, no workspace.
    assert lib.resa_rectify_workspace_size(1, 8, 32, 32768, 32768) == 0


def test_product_never_imports_oracle():
    """The library package must not reach the oracle (no CPU fallback)."""
    pkg = os.path.join(ROOT, "paper_2506_04108_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".cpp", ".hip", ".h")):
                text = open(os.path.join(dirpath, fn)).read()
                assert "import oracle" not in text and "from oracle" not in text, fn


@pytest.mark.parametrize("batch,heads,g", [(1, 1, 1), (2, 4, 7), (8, 8, 4)])
def test_step_workspace_keeps_flags_apart(batch, heads, g):
    """The step's workspace has room for the ready flags of the largest split
    count whatever the call's own, so no scratch of one call ever lies where
    another looks for a flag: sizes for 1 and 256 splits differ by the
    partials alone (lse and 128 floats a row, padded to 256 bytes)."""
    size = lambda s: L.lib().resa_step_workspace_size(batch, heads, heads * g, 6000, 16, 38, s)  # noqa: E731
    pad = lambda x: -(-x // 256) * 256  # noqa: E731
    rows = batch * heads * g
    assert size(256) - size(1) == pad(256 * rows * 4) - pad(rows * 4) + 255 * rows * 512


def test_workspace_sizes_grow_with_length():
    """A workspace sized for a longer context serves every shorter one: the
    selection, decode, fused-step and rectification sizes never decrease as
    the length (or the selected-block capacity) grows (lengths 65536 /
    65537 around the rectification's 128-key chunk minimum included), and
    the automatic split count stays in [1, 256] with at least one 16-token
    chunk per wave of four."""
    lib = L.lib()
    lengths = sorted(set([1, 15, 16, 17, 2047, 2048, 2049, 65536, 65537, 65600]
                         + [int(1.03 ** i) + 16 * (i % 7) for i in range(470)]))
    for batch, heads, g in ((1, 1, 1), (1, 8, 4), (2, 2, 7), (3, 4, 2), (8, 8, 4), (16, 8, 4), (64, 4, 8)):
        for b in (16, 32, 64):
            prev_sel = prev_step = 0
            for ln in lengths:
                sel = lib.resa_select_workspace_size(batch, heads, ln, b)
                assert sel >= prev_sel, (batch, heads, b, ln)
                prev_sel = sel
                m = -(-ln // b)
                n_cap = max(1, m // 10)
                step = lib.resa_step_workspace_size(batch, heads, heads * g, ln, b, n_cap, 0)
                assert step >= prev_step, (batch, heads, b, ln)
                prev_step = step
            prev_dec = 0
            for n_cap in range(1, 3000, 7):
                s = lib.resa_decode_num_splits(batch, heads, n_cap, b)
                chunks = n_cap * (b // 16)
                assert 1 <= s <= 256
                assert s == 1 or s <= chunks // 4, (batch, heads, n_cap, b, s)
                dec = lib.resa_decode_workspace_size(batch, heads, heads * g, n_cap, b, 0)
                assert dec >= prev_dec, (batch, heads, n_cap, b)
                prev_dec = dec
        for f in (1, 16, 32, 300):
            prev_rect = 0
            for ln in lengths:
                if ln < f:
                    continue
                r = lib.resa_rectify_workspace_size(batch, heads, heads * g, f, ln)
                assert r >= prev_rect, (batch, heads, g, f, ln)
                prev_rect = r
