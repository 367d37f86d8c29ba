"""GPU parity of decode calls that take both phases in one launch (dense attention; small clustered calls) at the edges of their
batches, chunks and of the rule that picks them.  Reference: the same attention in 64 bits."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W

import gpu_util as G

SCALE = float(np.float32(1 / math.sqrt(128)))
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
CODE = {"bf16": W.BF16, "f32": W.F32}


def _reference(q, kc, v, h2c, rep, T):
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for b in range(q.shape[0]):
        for h in range(q.shape[1]):
            c = int(h2c[b][h])
            p = torch.softmax(SCALE * (kc[b, c, :T].double() @ q[b, int(rep[b][c])].double()), 0)
            out[b, h] = p @ v[b, h, :T].double()
    return out


def _check(got, ref, dtype):
    assert bool(torch.isfinite(got).all())
    err = (got.double() - ref).abs().amax(-1) / ref.abs().amax(-1)
    assert float(err.max()) < (1e-5 if dtype == "f32" else 2e-5), float(err.max())       # fp32 sums, as for the other kernels


def _tensors(B, H, kk, T, cap, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, kc, v = (torch.randn(s, generator=g, device="cuda").to(DT[dtype]) for s in ((B, H, 128), (B, kk, cap, 128), (B, H, cap, 128)))
    kc[:, :, T:], v[:, :, T:] = float("nan"), float("nan")             # rows past the context are never read
    return q, kc, v


@pytest.mark.parametrize("dtype,B,H,kk,T", [
    ("bf16", 1, 1, 1, 1), ("bf16", 1, 5, 2, 31), ("bf16", 1, 5, 2, 33), ("f32", 1, 5, 2, 15), ("f32", 1, 5, 2, 17),   # one batch of keys
    ("bf16", 2, 7, 3, 255), ("bf16", 2, 7, 3, 257), ("f32", 2, 7, 3, 129), ("bf16", 1, 72, 16, 513),     # one round of the waves
    ("bf16", 1, 72, 16, 640), ("bf16", 1, 72, 16, 641), ("f32", 1, 72, 16, 320), ("f32", 1, 72, 16, 321),
    ("bf16", 1, 73, 9, 512), ("bf16", 1, 73, 9, 513), ("bf16", 4, 32, 8, 512), ("bf16", 3, 43, 8, 224), ("bf16", 3, 43, 8, 225),
    ("f32", 4, 64, 8, 112), ("f32", 4, 64, 8, 113), ("bf16", 1, 257, 8, 40), ("bf16", 2, 70, 69, 100),
])
def test_small_clustered_calls(dtype, B, H, kk, T):
    """Attention, and the same with the last row still to be appended; the first slot's representative stands for another slot
    as well, and the last slot of row 0 is unused."""
    print(f"[small decode] {dtype} B={B} H={H} k={kk} T={T}", flush=True)
    q, kc, v = _tensors(B, H, kk, T, T + 3, dtype, B + H + T)
    h2c, rep = W.random_membership(np.random.default_rng(T), B, H, kk)
    rep = rep.copy()
    if kk > 2:
        rep[:, 1] = rep[:, 0]
    hd, rd = torch.from_numpy(h2c).cuda(), torch.from_numpy(rep).cuda()
    ref = _reference(q, kc, v, h2c, rep, T)
    ws = G.poisoned_workspace(B, H, kk, T, 128, CODE[dtype])
    whole, out = G.guarded((B, H, 128), torch.float32, float("nan"))
    C.chai_decode_attention(q, kc, v, hd, rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    _check(out, ref, dtype)
    assert G.guards_intact(whole, (B, H, 128), float("nan"))

    k_new = torch.randn((B, H, 128), device="cuda").to(DT[dtype])
    for b in range(B):
        k_new[b, rep[b].tolist()] = kc[b, :, T - 1] if len(set(rep[b].tolist())) == kk else k_new[b, rep[b].tolist()]
        kc[b, :, T - 1] = k_new[b, rep[b].tolist()]
    ref = _reference(q, kc, v, h2c, rep, T)
    kc2, v2, v_new = kc.clone(), v.clone(), v[:, :, T - 1].clone()
    kc2[:, :, T - 1], v2[:, :, T - 1] = 9.0, 9.0
    if kk > 2:
        used = rep.copy()
        used[0, kk - 1] = -1
        rd = torch.from_numpy(used).cuda()
        kc[0, kk - 1, T - 1] = 9.0
    out.fill_(float("nan"))
    C.chai_decode_step(q, k_new, v_new, kc2, v2, hd, rd, T, SCALE, out, ws)
    torch.cuda.synchronize()
    live = torch.ones((B, H), dtype=torch.bool, device="cuda")
    if kk > 2:
        live[0] = hd[0] != kk - 1
    _check(out[live], ref[live], dtype)
    assert torch.equal(kc2.view(torch.uint8), kc.view(torch.uint8)) and torch.equal(v2.view(torch.uint8), v.view(torch.uint8))


@pytest.mark.parametrize("dtype,B,H,T", [
    ("bf16", 1, 1, 1), ("bf16", 1, 3, 40), ("f32", 1, 1, 40000),       # 128 chunks
    ("bf16", 1, 32, 700), ("bf16", 1, 32, 1024), ("bf16", 1, 32, 1025), ("f32", 1, 52, 2000),
    ("bf16", 2, 64, 513), ("bf16", 1, 129, 1), ("bf16", 3, 43, 300), ("bf16", 8, 32, 130), ("f32", 1, 256, 900),
    ("bf16", 1, 257, 799), ("bf16", 1, 257, 800), ("bf16", 1, 383, 801), ("bf16", 6, 64, 801), ("f32", 10, 50, 333),
    ("bf16", 1, 130, 12288), ("bf16", 1, 130, 12289),                  # the most tokens of a chunk
    ("bf16", 1, 128, 24577), ("bf16", 1, 256, 12289),                  # chunks doubled in number
    ("bf16", 1, 1, 1600000),                                           # more than the chunks hold: two launches
])
def test_dense_calls(dtype, B, H, T):
    print(f"[dense decode] {dtype} B={B} H={H} T={T}", flush=True)
    q, k, v = _tensors(B, H, H, T, T + 2, dtype, H + T)
    ident = np.tile(np.arange(H, dtype=np.int32), (B, 1))
    ws = G.poisoned_workspace(B, H, H, T, 128, CODE[dtype])
    whole, out = G.guarded((B, H, 128), torch.float32, float("nan"))
    C.chai_dense_decode_attention(q, k, v, T, SCALE, out, ws)
    torch.cuda.synchronize()
    _check(out, _reference(q, k, v, ident, ident, T), dtype)
    assert G.guards_intact(whole, (B, H, 128), float("nan"))
    o2 = torch.empty_like(out)
    C.chai_decode_attention(q, k, v, torch.from_numpy(ident).cuda(), torch.from_numpy(ident).cuda(), T, SCALE, o2, ws)
    torch.cuda.synchronize()
    assert torch.equal(out, o2)


@pytest.mark.parametrize("H,T", [(4, 100), (4, 2000), (300, 900)])
def test_large_scores_and_an_infinite_value(H, T):
    """Scores of some thousands (chunks whose maxima lie far apart), and an infinite value in the last row, whose padding
    is not weighed with it."""
    q, k, v = _tensors(1, H, H, T, T, "bf16", T)
    k *= 100
    ident = np.arange(H, dtype=np.int32)[None]
    ws = G.poisoned_workspace(1, H, H, T, 128, W.BF16)
    out = torch.empty((1, H, 128), device="cuda")
    C.chai_dense_decode_attention(q, k, v, T, SCALE, out, ws)
    ref = _reference(q, k, v, ident, ident, T)
    torch.cuda.synchronize()
    # a score of 10^3 to 10^4 carries 2^-24 of itself into the exponent
    assert float(((out.double() - ref).abs().amax(-1) / ref.abs().amax(-1)).max()) < 4e-3
    k /= 100
    v[:, :, T - 1, 7] = float("inf")
    C.chai_dense_decode_attention(q, k, v, T, SCALE, out, ws)
    torch.cuda.synchronize()
    assert bool((out[:, :, 7] == float("inf")).all()) and bool(torch.isfinite(out[:, :, :7]).all()) and bool(torch.isfinite(out[:, :, 8:]).all())


@pytest.mark.parametrize("dtype,H,T", [("bf16", 4, 100), ("f32", 4, 2000), ("bf16", 4, 12289), ("bf16", 300, 900)])
def test_values_near_the_largest_and_chunks_without_weight(dtype, H, T):
    """Sums of values that a float just holds stay finite, and keys that give -inf leave their tokens without weight, whole
    chunks of them too."""
    q, k, v = _tensors(1, H, H, T, T, dtype, T)
    q[..., 0] = 1.0
    k[:, :, : T // 2, 0] = -float("inf")
    v[..., 5] = -2e38
    ident = np.arange(H, dtype=np.int32)[None]
    out = torch.full((1, H, 128), float("nan"), device="cuda")
    C.chai_dense_decode_attention(q, k, v, T, SCALE, out, G.poisoned_workspace(1, H, H, T, 128, CODE[dtype]))
    torch.cuda.synchronize()
    ref = _reference(q, k, v, ident, ident, T)
    # column 5 by itself: next to it the others would be nothing
    _check(out[..., 5:6], ref[..., 5:6], dtype)
    others = [c for c in range(128) if c != 5]
    _check(out[..., others], ref[..., others], dtype)


@pytest.mark.parametrize("dtype,H,T", [("f32", 4, 256), ("bf16", 4, 300), ("f32", 4, 2000), ("bf16", 300, 900)])
def test_values_near_the_smallest(dtype, H, T):
    """Values of 2^-120, whose products with probabilities are denormal: a product of a weight and a value is off by 2^-150 at
    most, the T of them by T 2^-150, next to a result of at least 2^-120 T^-1/2."""
    q, k, v = _tensors(1, H, H, T, T, dtype, T)
    v = (v.double() * 2.0 ** -120).to(v.dtype)
    ident = np.arange(H, dtype=np.int32)[None]
    out = torch.full((1, H, 128), float("nan"), device="cuda")
    C.chai_dense_decode_attention(q, k, v, T, SCALE, out, G.poisoned_workspace(1, H, H, T, 128, CODE[dtype]))
    torch.cuda.synchronize()
    ref = _reference(q, k, v, ident, ident, T)
    err = (out.double() - ref).abs().amax(-1) / ref.abs().amax(-1)
    assert float(err.max()) < (1e-5 if dtype == "f32" else 2e-5) + T ** 1.5 * 2.0 ** -30, float(err.max())
