"""GPU parity of the decode calls at the lines where the launch plan changes (streams taken whole in column halves or split
over tokens, 64-token score chunks, 8-bit rows in workgroups of four or eight waves), and of k-means at the edges of its
lane groups and masks, against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W
from oracle import chai_oracle as O

import gpu_util as G
from gpu_util import dev
from test_gpu_q8 import _run_case

SCALE = float(np.float32(1 / math.sqrt(128)))


@pytest.mark.parametrize("dtype,B,H,kk,T", [
    (W.BF16, 2, 40, 4, 1536), (W.BF16, 2, 40, 4, 1537), (W.F32, 2, 40, 4, 768), (W.F32, 2, 40, 4, 769),   # whole / split
    (W.BF16, 12, 16, 5, 1300), (W.F32, 12, 16, 5, 1300),                                                  # 192 heads
    (W.BF16, 16, 8, 4, 256), (W.BF16, 13, 8, 5, 256),                      # 64 and 65 score workgroups of 256 tokens
    (W.BF16, 1, 8, 3, 1), (W.F32, 1, 8, 3, 63), (W.BF16, 1, 8, 3, 64), (W.F32, 1, 8, 3, 65), (W.BF16, 1, 8, 8, 1025),
    (W.BF16, 1, 4, 2, 2200),                                               # 18 partial rows: more than one batch of requests
])
def test_decode_and_step_at_plan_edges(dtype, B, H, kk, T):
    """chai_decode_attention, chai_decode_step (last row appended) and the shared-value form against the oracle."""
    print(f"[plan] dtype={dtype} B={B} H={H} k={kk} T={T}", flush=True)
    g = np.random.default_rng(T + B)
    rtol = 1e-5 if dtype == W.F32 else 2e-5
    h2c, rep = W.random_membership(g, B, H, kk)
    q, k, v = W.normal(g, (B, H, 128), dtype), W.normal(g, (B, H, T, 128), dtype), W.normal(g, (B, H, T, 128), dtype)
    ref = O.clustered_decode(q, k, v, h2c, rep, T, SCALE)
    kd, vd, hd, rd = dev(k), dev(v), dev(h2c), dev(rep)
    kc = torch.zeros((B, kk, T, 128), dtype=kd.dtype, device="cuda")
    C.chai_compact_kcache(kd, rd, kc, T)
    ws = G.poisoned_workspace(B, H, kk, T, 128, dtype)
    out = torch.full((B, H, 128), float("nan"), dtype=torch.float32, device="cuda")
    C.chai_decode_attention(dev(q), kc, vd, hd, rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    ok, worst = G.rows_close(out.cpu().numpy(), ref, rtol)
    assert ok, worst
    # the same with the last row still to be appended
    k_new, v_new, kc2, vd2 = kd[:, :, T - 1].contiguous(), vd[:, :, T - 1].contiguous(), kc.clone(), vd.clone()
    kc2[:, :, T - 1], vd2[:, :, T - 1] = 9.0, 9.0
    out.fill_(float("nan"))
    C.chai_decode_step(dev(q), k_new, v_new, kc2, vd2, hd, rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    ok, worst = G.rows_close(out.cpu().numpy(), ref, rtol)
    assert ok and torch.equal(kc2, kc) and torch.equal(vd2, vd), worst
    vc = torch.zeros_like(kc)
    C.chai_compact_kcache(vd, rd, vc, T)
    C.chai_decode_attention_shared_v(dev(q), kc, vc, hd, rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    ok, worst = G.rows_close(out.cpu().numpy(), O.shared_v_decode(q, k, v, h2c, rep, T, SCALE), rtol)
    assert ok, worst


@pytest.mark.parametrize("B,H,kk,T", [(2, 32, 4, 1536), (2, 32, 4, 1537), (1, 6, 3, 1600), (4, 72, 8, 2050)])
def test_decode_q8_at_plan_edges(B, H, kk, T):
    _run_case(8100 + T, B, H, kk, T, T + 1, W.BF16)


@pytest.mark.parametrize("H,F,k", [(1, 25, 1), (2, 1, 2), (31, 25, 3), (32, 32, 16), (33, 33, 17), (64, 25, 16), (65, 25, 16),
                                   (72, 25, 72), (128, 4, 9), (129, 64, 8), (256, 25, 5), (256, 22, 256), (200, 3, 150)])
@pytest.mark.parametrize("levels", [0, 2])
def test_kmeans_bit_exact_at_lane_group_edges(H, F, k, levels):
    """levels = 2: features of few values, so that distances tie and centres run empty (the repair path)."""
    g = np.random.default_rng(H * 7 + F * 3 + k + levels)
    B = 3
    feat = (g.integers(0, levels, (B, H, F)) if levels else g.random((B, H, F))).astype(np.float32)
    init = np.stack([g.choice(H, size=k, replace=False) for _ in range(B)]).astype(np.int32)
    for max_iter in (1, 50):
        got = C.chai_assign_clusters(dev(feat), dev(init), max_iter)
        torch.cuda.synchronize()
        want = O.kmeans(feat, init, max_iter=max_iter)
        for a, b in zip(got, want):
            assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("n_tok", [1, 5, 8])
@pytest.mark.parametrize("dtype", [W.BF16, W.F32])
def test_features_of_every_prompt_length(n_tok, dtype):
    g = np.random.default_rng(n_tok)
    q, k = W.normal(g, (2, 7, n_tok, 128), dtype), W.normal(g, (2, 7, n_tok + 1, 128), dtype)
    feat = torch.full((2, 7, n_tok * n_tok), float("nan"), dtype=torch.float32, device="cuda")
    C.chai_score_features(dev(q), dev(k), n_tok, SCALE, feat)
    torch.cuda.synchronize()
    s = SCALE * np.einsum("bhid,bhjd->bhij", W.as_f64(q), W.as_f64(k)[:, :, :n_tok])
    s = np.where(np.tril(np.ones((n_tok, n_tok), bool)), s, -np.inf)
    e = np.exp(s - s.max(-1, keepdims=True))
    want = (e / e.sum(-1, keepdims=True)).reshape(2, 7, -1)
    # one rounding to fp32 of a value that 64 bits carry to a few 1e-15
    assert np.all(np.abs(feat.cpu().numpy() - want) <= 2.0 ** -24 * want + 1e-14)


@pytest.mark.parametrize("score_dtype,value_dtype", [(W.F32, W.BF16), (W.BF16, W.F32)])
@pytest.mark.parametrize("B,H,kk,T", [(1, 32, 8, 1024), (1, 8, 3, 769), (1, 8, 3, 768), (1, 12, 4, 1536), (2, 100, 2, 1400)])
def test_phases_of_different_types_agree_on_the_workspace(score_dtype, value_dtype, B, H, kk, T):
    """The two phase calls with queries and keys of one type and values of the other: the layout between them does not
    depend on the type."""
    print(f"[mixed] {score_dtype}->{value_dtype} B={B} H={H} k={kk} T={T}", flush=True)
    g = np.random.default_rng(T + H)
    h2c, rep = W.random_membership(g, B, H, kk)
    # bf16 numbers, so that the oracle can be given all of them in fp32
    q, k, v = (W.as_f64(W.normal(g, s, W.BF16)).astype(np.float32) for s in ((B, H, 128), (B, H, T, 128), (B, H, T, 128)))
    ref = O.clustered_decode(q, k, v, h2c, rep, T, SCALE)
    tt = {W.F32: torch.float32, W.BF16: torch.bfloat16}
    kd, hd, rd = dev(k).to(tt[score_dtype]), dev(h2c), dev(rep)
    kc = torch.zeros((B, kk, T, 128), dtype=kd.dtype, device="cuda")
    C.chai_compact_kcache(kd, rd, kc, T)
    ws = G.poisoned_workspace(B, H, kk, T, 128, W.F32)
    out = torch.full((B, H, 128), float("nan"), dtype=torch.float32, device="cuda")
    C.chai_decode_scores(dev(q).to(tt[score_dtype]), kc, rd, T, SCALE, ws)
    C.chai_decode_values(dev(v).to(tt[value_dtype]), hd, rd, T, out, ws)
    torch.cuda.synchronize()
    ok, worst = G.rows_close(out.cpu().numpy(), ref, 2e-5)
    assert ok, worst


@pytest.mark.parametrize("H,F,k,bad", [(32, 25, 8, (2,)), (32, 25, 8, (0,)), (72, 25, 16, (2, 5)), (40, 40, 12, (3, 9)),
                                       (33, 3, 1, (0,)), (24, 9, 24, (1, 6, 22))])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_kmeans_with_features_that_are_not_finite(H, F, k, bad, value):
    """Heads whose features are NaN or infinite are starting centres `bad`: the distances to them are NaN, which an ascending
    scan passes by (or keeps, if it met it first)."""
    g = np.random.default_rng(H + F + k)
    B = 2
    feat = g.random((B, H, F)).astype(np.float32)
    init = np.stack([g.choice(H, size=k, replace=False) for _ in range(B)]).astype(np.int32)
    for b in range(B):
        for j in bad:
            feat[b, init[b, j], :: 2] = value
    for max_iter in (1, 2, 50):
        got = C.chai_assign_clusters(dev(feat), dev(init), max_iter)
        torch.cuda.synchronize()
        want = O.kmeans(feat, init, max_iter=max_iter)
        for a, b in zip(got, want):
            assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("dtype,B,H,kk,T", [
    (W.BF16, 6, 12, 8, 384), (W.BF16, 6, 12, 8, 385), (W.BF16, 7, 9, 7, 385), (W.BF16, 1, 6, 4, 1537),     # 48, 49 streams
    (W.F32, 6, 12, 8, 384), (W.F32, 1, 6, 4, 385), (W.F32, 7, 9, 7, 385), (W.BF16, 4, 72, 16, 1100), (W.F32, 1, 3, 1, 129)])
def test_shared_values_at_plan_edges(dtype, B, H, kk, T):
    """Few shared streams: whole up to 384 tokens, split beyond; more than 48 streams as every other call."""
    print(f"[shared] dtype={dtype} B={B} H={H} k={kk} T={T}", flush=True)
    g = np.random.default_rng(T + B)
    h2c, rep = W.random_membership(g, B, H, kk)
    q, k, v = W.normal(g, (B, H, 128), dtype), W.normal(g, (B, H, T, 128), dtype), W.normal(g, (B, H, T, 128), dtype)
    kd, rd = dev(k), dev(rep)
    kc = torch.zeros((B, kk, T, 128), dtype=kd.dtype, device="cuda")
    vc = torch.zeros_like(kc)
    C.chai_compact_kcache(kd, rd, kc, T)
    C.chai_compact_kcache(dev(v), rd, vc, T)
    ws = G.poisoned_workspace(B, H, kk, T, 128, dtype)
    out = torch.full((B, H, 128), float("nan"), dtype=torch.float32, device="cuda")
    C.chai_decode_attention_shared_v(dev(q), kc, vc, dev(h2c), rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    ok, worst = G.rows_close(out.cpu().numpy(), O.shared_v_decode(q, k, v, h2c, rep, T, SCALE), 1e-5 if dtype == W.F32 else 2e-5)
    assert ok, worst
