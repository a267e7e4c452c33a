"""V values over the whole range of bf16 in the rectification: finite results
for every finite V, also through the merge of the splits, and every row bounded
by the values that the row itself can see."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, up

pytestmark = pytest.mark.gpu
TOL = 1.2e-3  # weights rounded to fp16: 2^-12, of a largest |V| below 4.9


def rectify(B, H, g, f, L, plants, tag):
    """dense_rectify of the last f of L rows, N(0, 1) inputs with `plants`
    (row or slice, dim, value) put into every group's V. Returns the groups'
    worst error, each output entry's scaled by max(1, largest |V_d| the row
    sees), over the first and the last group."""
    w = W.TINY_4K.with_(batch=B, num_kv_heads=H, num_q_heads=H * g, seq_len=L, seed_tag=tag)
    K, V = W.kv_cache(w, capacity=-(-L // 16) * 16)
    V = V.copy()
    for row, d, x in plants:
        V[:, :, row, d] = W.f32_to_bf16_bits(np.array([x], np.float32))[0]
    cache = make_cache(K, V, 16, sentinel=False)
    lt = i32([L] * B)
    R.block_summarize(cache, lt)
    kf, vf = np.ascontiguousarray(K[:, :, L - f:L]), np.ascontiguousarray(V[:, :, L - f:L])
    qf = W.rectify_inputs(w, 9, kf, vf, f)[0]
    out, _ = R.dense_rectify(cache, up(qf), up(kf), up(vf), lt, L)
    torch.cuda.synchronize()
    go = out.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(go)), "non-finite rectify output"
    worst = 0.0
    for bi, hi in {(0, 0), (B - 1, H - 1)}:
        Kg, Vg = O.bf16_to_f64(K[bi, hi, :L]), O.bf16_to_f64(V[bi, hi, :L])
        seen = np.maximum.accumulate(np.abs(Vg), axis=0)
        for r in range(f):
            n = L - f + r + 1
            o, _ = O.attend(O.bf16_to_f64(qf[bi, hi * g:(hi + 1) * g, r]), Kg, Vg, np.arange(n), w.sm_scale)
            err = np.abs(go[bi, hi * g:(hi + 1) * g, r] - o) / np.maximum(1.0, seen[n - 1])
            worst = max(worst, float(err.max()))
    print(f"V range B={B} H={H} g={g} f={f} L={L} {tag}: worst {worst:.2e}", flush=True)
    return worst


@pytest.mark.parametrize("B,H,g,f,L", [(1, 2, 1, 8, 2000),     # 4 waves, 16 splits
                                       (1, 2, 1, 8, 3000),     # more than 16
                                       (8, 4, 1, 129, 2000)])  # 8 waves, 8 splits
def test_merge_of_the_largest_values(B, H, g, f, L):
    """Whole dimensions of +-3e38: every split's row is close to the largest
    float, and so is their mean."""
    assert rectify(B, H, g, f, L, [(slice(None), 5, 3e38), (slice(None), 77, -3.3e38)], "largest") <= TOL
