"""One decode-step workspace over calls of other lengths, selected counts and
split counts, up and down: what the step keeps between calls must not move
with them. Checked against resa_append_select + resa_sparse_decode on fresh
workspaces."""
import dataclasses

import pytest
import torch

import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, up

pytestmark = pytest.mark.gpu


def copy_of(cache):
    return dataclasses.replace(cache, **{f: getattr(cache, f).clone() for f in ("k", "v", "kmin", "kmax")})


@pytest.mark.parametrize("g", [3, 4])
def test_lengths_up_and_down(g):
    B, H, cap = 2, 4, 1280
    w = W.LONG_64K.with_(batch=B, num_kv_heads=H, num_q_heads=H * g, seq_len=1200, seed_tag=f"stepws{g}")
    K, V = W.kv_cache(w, capacity=cap)
    cache = make_cache(K, V, 16, sentinel=False)
    R.block_summarize(cache, i32([1200, 1100]))
    ref = copy_of(cache)
    ws = R.Workspace()
    # Sized once for the longest call, the largest count and split count.
    ws.get(max(R.lib().resa_step_workspace_size(B, H, H * g, cap - 1, 16, 80, s) for s in (0, 1, 5, 24)))
    size = ws.buf.numel()
    calls = [(1200, 64, 0), (300, 20, 0), (1216, 64, 0), (1201, 76, 24), (40, 4, 1), (1233, 77, 0), (700, 44, 5),
             (1200, 64, 0), (16, 2, 24), (1250, 79, 0)]
    for step, (L, n, splits) in enumerate(calls * 3):
        kn, vn = (up(x) for x in W.decode_kv(w, step % 7))
        q = up(W.decode_query(w, step % 5))
        l1, l2 = i32([L, L - 7]), i32([L, L - 7])
        idx, ns, out, lse = R.decode_step(cache, kn, vn, q, l1, L, 1.0, n, 1, n_cap=n, num_splits=splits,
                                          workspace=ws)
        ri, rn = R.append_select(ref, kn, vn, q, l2, L, 1.0, n, 1, n_cap=n)
        ro, rl = R.sparse_decode(ref, q, l2, ri, rn, num_splits=splits)
        torch.cuda.synchronize()
        assert ws.buf.numel() == size
        assert torch.equal(l1, l2) and torch.equal(ns, rn) and torch.equal(idx, ri), (step, L)
        assert torch.equal(out, ro) and torch.equal(lse, rl), (step, L)
    for f in ("k", "v", "kmin", "kmax"):
        assert torch.equal(getattr(cache, f), getattr(ref, f)), f
