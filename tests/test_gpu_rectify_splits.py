"""Split counts of long windows over short and longer caches, from one split to
as many as fill the chip, with and without a sequence mask, against the oracle
on two groups: one workspace of exactly the size asked for at the largest
length serves every shorter call.

Bound: weights rounded to fp16 (2^-12; below 2^-14 of the softmax reference by
2^-25 of it) times the largest |V| (below 4.9)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, up
from oracle.compare import max_abs_err
from paper_2506_04108_amd import _lib

pytestmark = pytest.mark.gpu
TOL = 1.2e-3


@pytest.mark.parametrize("B,H,g,f", [(1, 1, 1, 129),    # 1 workgroup per split
                                     (4, 2, 4, 50),     # 8
                                     (8, 4, 4, 40),     # 32
                                     (8, 8, 4, 64),     # 64
                                     (12, 8, 1, 130),   # 96
                                     (5, 8, 2, 500)])   # 160, four query blocks
@pytest.mark.parametrize("masked", [False, True])
def test_splits(B, H, g, f, masked):
    lengths = [260, 512, 577, 700, 1200, 2053] if f < 260 else [517, 900, 1300]
    w = W.TINY_4K.with_(batch=1, num_kv_heads=H, num_q_heads=H * g, seq_len=max(lengths), seed_tag=f"splits{B}{H}{g}")
    cap = -(-max(lengths) // 16) * 16
    K1, V1 = W.kv_cache(w, capacity=cap)
    K = np.stack([np.roll(K1[0], i, axis=0) for i in range(B)])
    V = np.stack([np.roll(V1[0], i, axis=1) for i in range(B)])
    q1 = W.rectify_inputs(w, 4, K1[:, :, :f], V1[:, :, :f], f)[0]
    qf = np.stack([np.roll(q1[0], i, axis=1) for i in range(B)])
    size = _lib.lib().resa_rectify_workspace_size(B, H, H * g, f, max(lengths))
    ws = R.Workspace()
    assert ws.get(size).numel() == max(size, 256)
    mask = i32([(i + 1) % 2 for i in range(B)]) if masked else None
    last = (B - 1) // 2 * 2 if masked else B - 1
    for L in lengths:
        cache = make_cache(K, V, 16, sentinel=False)
        kf, vf = np.ascontiguousarray(K[:, :, L - f:L]), np.ascontiguousarray(V[:, :, L - f:L])
        out = torch.full((B, H * g, f, 128), 7.0, device="cuda")
        out, lse = R.dense_rectify(cache, up(qf), up(kf), up(vf), i32([L] * B), L, out=out, workspace=ws, seq_mask=mask)
        torch.cuda.synchronize()
        go, gl = out.cpu().numpy(), lse.cpu().numpy()
        if masked:
            assert np.all(go[1::2] == 7.0)
        for bi, hi in {(0, 0), (last, H - 1)}:
            Kg, Vg = O.bf16_to_f64(K[bi, hi]), O.bf16_to_f64(V[bi, hi])
            kmin, kmax = O.block_summaries(Kg, L, 16)
            sl = slice(hi * g, (hi + 1) * g)
            ro, rl = O.rectify_group(O.bf16_to_f64(qf[bi, sl]), Kg, Vg, kmin, kmax, L, f, 16, w.sm_scale,
                                     Kg[L - f:L].copy(), Vg[L - f:L].copy())
            eo, el = max_abs_err(go[bi, sl], ro), max_abs_err(gl[bi, sl], rl)
            print(f"splits B={B} H={H} g={g} f={f} L={L} masked={masked} ({bi},{hi}): |dO| {eo:.2e} |dlse| {el:.2e}",
                  flush=True)
            assert eo <= TOL and el <= 1e-4
    assert ws.buf.numel() == max(size, 256)  # never grown
