"""Rectification at the edges of its tiles and of its workgroup choice,
against the oracle: windows of 1 .. 129 and 255 .. 777 rows (4 and 8 waves, one
to four query blocks a group, each a workgroup of its own; two blocks a
workgroup are test_gpu_rectify_pairs.py's), lengths around the 32- and 64-key
tiles and the splits' ends, both layouts, and logits that climb along the
sequence (the softmax reference has to move).

Bound: a weight is rounded to fp16, by 2^-12 of itself from 2^-14 of the softmax
reference on and by at most 2^-25 of the reference below (fp16's subnormals),
and the weights sum to at least the reference. An output is off by at most
2^-12 of its dimension's largest |V| (below 4.9 here), 1.2e-3, and by 2^-25 of
it for every key of such a small weight (3e-4 if all of 2000 were): rounding
errors of both signs stay far below the first term alone."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, make_paged_cache, up
from oracle.compare import max_abs_err

pytestmark = pytest.mark.gpu
TOL = 1.2e-3


def run(g, f, lens, paged=False, climb=0.0, tag="shape"):
    B, H, cap = len(lens), 2, -(-max(lens) // 64) * 64
    w = W.TINY_4K.with_(batch=B, num_kv_heads=H, num_q_heads=H * g, seq_len=max(lens), seed_tag=f"{tag}{g}-{f}")
    K, V = W.kv_cache(w, capacity=cap)
    base = lambda X: np.stack([X[i, :, lens[i] - f:lens[i]] for i in range(B)])  # noqa: E731
    qf, kf, vf = W.rectify_inputs(w, 1, base(K), base(V), f)
    if climb:  # logits rise by climb * 8 / sqrt(128) over the sequence, every row alike
        rise = np.zeros((cap, 128), np.float32)
        rise[:, 7] = np.linspace(0.0, climb, cap)
        K = W.f32_to_bf16_bits(W.bf16_bits_to_f32(K) + rise)
        kf = np.stack([W.f32_to_bf16_bits(W.bf16_bits_to_f32(kf[i]) + rise[lens[i] - f:lens[i]]) for i in range(B)])
        q = W.bf16_bits_to_f32(qf).copy()
        q[..., 7] = 8.0
        qf = W.f32_to_bf16_bits(q)
    cache = make_paged_cache(K, V, 16, lens, seed=5, sentinel=False) if paged else make_cache(K, V, 16, sentinel=False)
    lt = i32(lens)
    R.block_summarize(cache, lt)
    out, lse = R.dense_rectify(cache, up(qf), up(kf), up(vf), lt, max(lens))
    torch.cuda.synchronize()
    st = O.DecodeState(O.bf16_to_f64(K), O.bf16_to_f64(V), list(lens), 16)
    ro, rl = st.rectify(O.bf16_to_f64(qf), O.bf16_to_f64(kf), O.bf16_to_f64(vf), f, w.sm_scale)
    eo, el = max_abs_err(out.cpu().numpy(), ro), max_abs_err(lse.cpu().numpy(), rl)
    print(f"rectify g={g} f={f} lens={lens} paged={paged} climb={climb}: |dO| {eo:.2e} |dlse| {el:.2e}", flush=True)
    assert eo <= TOL and el <= 1e-4


@pytest.mark.parametrize("g,f", [(1, 1), (1, 127), (1, 128), (1, 129), (3, 43), (8, 16), (1, 255), (1, 256), (1, 257),
                                 (2, 128), (1, 513), (4, 193), (7, 111)])
@pytest.mark.parametrize("paged", [False, True])
def test_row_counts(g, f, paged):
    run(g, f, [f + 70, f + 3], paged)


@pytest.mark.parametrize("f", [32, 129])
@pytest.mark.parametrize("L", [129, 159, 160, 161, 191, 192, 193, 255, 256, 257, 321, 449])
def test_lengths(f, L):
    run(2, f, [L, max(f, L - 33)])


@pytest.mark.parametrize("g,f", [(4, 32), (4, 100), (1, 300)])
@pytest.mark.parametrize("climb", [15.0, 60.0, -60.0])
def test_climbing_logits(g, f, climb):
    """Logits rising by 15 and by 61 bits over the sequence (far outside fp16
    from the first tile's maximum) and falling by 61."""
    run(g, f, [2000, 1203], climb=climb, tag="climb")
