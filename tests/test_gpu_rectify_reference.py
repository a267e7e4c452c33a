"""The softmax reference of the rectification: where it is taken, that it is
found again after a tile without a finite score, and softmax scales of every
sign. Against the oracle, with logits that are set key by key."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2506_04108_amd as R
import workloads as W
from gpu_util import i32, make_cache, up
from oracle.compare import max_abs_err

pytestmark = pytest.mark.gpu


def rectify(K, V, q, f, sm_scale):
    """The last f rows of K and V, written again, and the oracle's result for
    query rows q [B, Hq, f, 128]; all bf16 bits."""
    L = K.shape[2]
    cache = make_cache(K, V, 16, sentinel=False)
    lt = i32([L] * K.shape[0])
    R.block_summarize(cache, lt)
    kf, vf = np.ascontiguousarray(K[:, :, L - f:]), np.ascontiguousarray(V[:, :, L - f:])
    out, lse = R.dense_rectify(cache, up(q), up(kf), up(vf), lt, L, sm_scale=sm_scale)
    torch.cuda.synchronize()
    st = O.DecodeState(O.bf16_to_f64(K), O.bf16_to_f64(V), [L] * K.shape[0], 16)
    ro, rl = st.rectify(O.bf16_to_f64(q), O.bf16_to_f64(kf), O.bf16_to_f64(vf), f, sm_scale)
    return out.cpu().numpy(), lse.cpu().numpy(), ro, rl


def test_reference_taken_again_within_a_split():
    """32 groups of 129 rows over 2048 keys: 8 splits of 256 keys, the
    reference taken every 128. One key a group, at the second range of a
    split, carries nearly all of the weight, 1024.4 times that of the range
    before it: against that range's reference it is rounded to 1024 (3.9e-4
    off), against its own it is exactly 1. Bound: fp32 rounding (2e-6)."""
    B, H, f, L = 8, 4, 129, 2048
    K = np.zeros((B, H, L, 128), np.float32)
    V = np.zeros((B, H, L, 128), np.float32)
    q = np.zeros((B, H, f, 128), np.float32)
    q[..., :2] = 1.0
    K[..., 0] = -10.0
    y = np.log(1024.4)
    y0 = float(W.bf16_bits_to_f32(W.f32_to_bf16_bits(np.array([y], np.float32)))[0])
    for bi in range(B):
        for hi in range(H):
            at = 256 * ((4 * bi + hi) % 7)
            K[bi, hi, at + 3, 0] = 0.0
            K[bi, hi, at + 128 + 7 * hi, :2] = y0, y - y0
            V[bi, hi, at + 128 + 7 * hi] = 1.0
    go, gl, ro, rl = rectify(*(W.f32_to_bf16_bits(x) for x in (K, V, q)), f, 1.0)
    eo, el = max_abs_err(go, ro), max_abs_err(gl, rl)
    print(f"reference within a split: |dO| {eo:.2e} |dlse| {el:.2e}", flush=True)
    assert eo <= 2e-6 and el <= 1e-5


@pytest.mark.parametrize("g,f", [(1, 8), (4, 32), (8, 17), (2, 200)])
def test_first_tile_without_a_finite_score(g, f):
    """Every second 64-key stretch scores -inf (the products overflow), so
    most splits begin with a tile that has no finite score; the other keys'
    logits are -40 (57 bits below zero). Bound: weights rounded to fp16
    (2^-12) times the largest |V| (below 4.9)."""
    B, H, L = 2, 2, 1500
    w = W.TINY_4K.with_(batch=B, num_kv_heads=H, num_q_heads=H * g, seq_len=L, seed_tag=f"inf{g}-{f}")
    V = W.kv_cache(w, capacity=1536)[1][:, :, :L + 4]
    K = np.zeros((B, H, L + 4, 128), np.float32)
    K[..., 1] = -40.0
    K[..., 0] = np.where(np.arange(L + 4) % 128 < 64, -3e38, 0.0)
    q = np.zeros((B, H * g, f, 128), np.float32)
    q[..., 0], q[..., 1] = 1e30, 1.0
    go, gl, ro, rl = rectify(W.f32_to_bf16_bits(K), V, W.f32_to_bf16_bits(q), f, 1.0)
    eo, el = max_abs_err(go, ro), max_abs_err(gl, rl)
    print(f"first tile -inf g={g} f={f}: |dO| {eo:.2e} |dlse| {el:.2e}", flush=True)
    assert eo <= 1.2e-3 and el <= 1e-4


@pytest.mark.parametrize("sm_scale", [0.0, -0.05, -0.6])
@pytest.mark.parametrize("g,f", [(4, 32), (4, 65)])
def test_softmax_scale_of_every_sign(g, f, sm_scale):
    """Zero and negative softmax scales, which the other calls take too: zero
    weighs every visible key alike, a negative one prefers the smallest
    products. Same bound as above."""
    B, H, L = 2, 2, 1008
    w = W.TINY_4K.with_(batch=B, num_kv_heads=H, num_q_heads=H * g, seq_len=L, seed_tag=f"sign{f}")
    K, V = (np.ascontiguousarray(x[:, :, :L]) for x in W.kv_cache(w, capacity=1024))
    q = W.rectify_inputs(w, 1, K[:, :, L - f:], V[:, :, L - f:], f)[0]
    go, gl, ro, rl = rectify(K, V, q, f, sm_scale)
    eo, el = max_abs_err(go, ro), max_abs_err(gl, rl)
    print(f"sm_scale {sm_scale} g={g} f={f}: |dO| {eo:.2e} |dlse| {el:.2e}", flush=True)
    assert eo <= 1.2e-3 and el <= 1e-4
