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


@pytest.mark.parametrize("B,H,g,f,L", [(1, 2, 4, 32, 1100),     # 4 waves, several splits
                                       (1, 2, 1, 100, 100),     # 4 waves, one split
                                       (2, 2, 4, 300, 900),     # 8 waves, several splits
                                       (8, 8, 4, 513, 520)])    # 8 waves, pairs of query blocks
def test_rows_before_a_large_value(B, H, g, f, L):
    """Values above the fp16 range at rows of the window that most query rows
    do not see: those keep the precision of the values they see, also where
    the large value sits in their own tile, and later rows stay within the
    bound of what they see. Several magnitudes in one dimension, and a
    dimension whose large value lies in the cache before the window."""
    r = L - f
    plants = [(r + f // 2, 5, 3e38), (r + f // 3, 6, 1e5), (r + 2 * f // 3, 6, -2e20), (L - 1, 7, 3e38),
              (r + 1, 40, 7e4), (r + 5, 40, -5e30), (r + f // 2 + 1, 41, 2.0 ** 36), (L - 3, 42, -1e9),
              (r + f // 2, 5 + 64, -65536.0), (r + f // 2 + 2, 100, 65280.0)]
    if r > 70:
        plants += [(64, 90, 8e4), (r - 1, 91, -3e38)]
    assert rectify(B, H, g, f, L, plants, "late") <= TOL
