"""Selection of short groups (one workgroup selects a whole group in LDS up to
320 blocks) at its edges, against the oracle: one block to 321, ragged
batches, exact ties, negative and equal scores, repeated calls on one
workspace (window hint set, then moved away by other queries), and the fused
append's rows, summaries and lengths."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, up
from oracle.compare import check_selection

pytestmark = pytest.mark.gpu


def scores_of(K64, L, b, q64):
    kmin, kmax = O.block_summaries(K64, L, b)
    return O.block_scores(O.pooled_query(q64), kmin, kmax)


@pytest.mark.parametrize("M", [1, 2, 15, 63, 64, 65, 127, 200, 256, 257, 319, 320, 321])
@pytest.mark.parametrize("n_local,sparsity", [(1, 0.9), (0, 0.5), (3, 0.95)])
def test_edges(M, n_local, sparsity):
    b, g, H = 16, 4, 2
    lens = [16 * M - 3, max(1, 16 * (M // 2) + 5), 1]
    cap = 16 * (M + 1)
    w = W.TINY_4K.with_(batch=3, num_kv_heads=H, num_q_heads=H * g, seq_len=max(lens), seed_tag=f"small{M}")
    K, V = W.kv_cache(w, capacity=cap)
    K64 = O.bf16_to_f64(K)
    cache = make_cache(K, V, b, sentinel=False)
    lt = i32(lens)
    R.block_summarize(cache, lt)
    ws = R.Workspace()
    for step in range(4):  # the last query points the other way: the hint misses
        q = W.decode_query(w, step)
        if step == 3:
            q = W.f32_to_bf16_bits(-4.0 * W.bf16_bits_to_f32(q))
        idx, ns = R.select_blocks(cache, up(q), lt, max(lens), sparsity, 2, n_local, workspace=ws)
        torch.cuda.synchronize()
        gi, gn, q64 = idx.cpu().numpy(), ns.cpu().numpy(), O.split_heads(O.bf16_to_f64(q)[:, :, None], H)[..., 0, :]
        for bi in range(3):
            m = O.num_blocks(lens[bi], b)
            n = O.num_selected(m, sparsity, 2, n_local)
            for hi in range(H):
                assert gn[bi, hi] == n
                s = scores_of(K64[bi, hi], lens[bi], b, q64[bi, hi])
                ids = gi[bi, hi, :n]
                assert np.all(np.diff(ids) > 0) and np.all(gi[bi, hi, n:] == -1)
                check_selection(ids, O.select_blocks(s, n, n_local), s, n, n_local)


@pytest.mark.parametrize("M,n", [(100, 30), (256, 128), (320, 128), (320, 1), (250, 249)])
@pytest.mark.parametrize("value", [0.0, 1.5, -2.0])
def test_ties_keep_the_lower_ids(M, n, value):
    """All blocks alike: equal scores go to the lower ids (and the local block)."""
    K = np.full((1, 1, 16 * M, 128), 0, np.uint16)
    K[...] = W.f32_to_bf16_bits(np.array([value], np.float32))[0]
    cache = make_cache(K, K, 16, sentinel=False)
    lt = i32([16 * M])
    R.block_summarize(cache, lt)
    q = torch.ones((1, 4, 128), dtype=torch.bfloat16, device="cuda")
    ws = R.Workspace()
    for _ in range(2):
        idx, ns = R.select_blocks(cache, q, lt, 16 * M, 1.0, n, 1, workspace=ws)
        torch.cuda.synchronize()
        assert ns.item() == n
        assert idx[0, 0].tolist() == list(range(n - 1)) + [M - 1]


@pytest.mark.parametrize("L", [15, 16, 319 * 16 + 15, 319 * 16 + 16])
def test_fused_append_matches_separate(L):
    """append_select on both sides of the 320-block border against append_kv
    and select_blocks: selections, lengths, rows and summaries bit for bit."""
    w = W.TINY_4K.with_(batch=2, num_kv_heads=2, num_q_heads=8, seq_len=L, seed_tag=f"smallapp{L}")
    cap = 16 * 322
    K, V = W.kv_cache(w, capacity=cap)
    c1, c2 = make_cache(K, V, 16, sentinel=False), make_cache(K, V, 16, sentinel=False)
    l1, l2 = i32([L, max(1, L // 3)]), i32([L, max(1, L // 3)])
    R.block_summarize(c1, l1)
    R.block_summarize(c2, l2)
    w1, w2 = R.Workspace(), R.Workspace()
    for step in range(3):
        kn, vn = W.decode_kv(w, step)
        q = up(W.decode_query(w, step))
        i1, n1 = R.append_select(c1, up(kn), up(vn), q, l1, L + step, 0.9, 4, 1, workspace=w1)
        R.append_kv(c2, up(kn), up(vn), l2, L + step)
        i2, n2 = R.select_blocks(c2, q, l2, L + step + 1, 0.9, 4, 1, workspace=w2)
        torch.cuda.synchronize()
        assert torch.equal(l1, l2) and torch.equal(n1, n2) and torch.equal(i1, i2)
    for f in ("k", "v", "kmin", "kmax"):
        assert torch.equal(getattr(c1, f), getattr(c2, f)), f
