"""GPU parity of the prefill kernel at the edges of its tiles and of the rules that number its workgroups: 128-row tiles
(small launches) and 256-row tiles, pairs and single tiles, more batch rows than one wave counts, unused cluster slots,
a running maximum that keeps moving."""
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
from test_gpu_prefill import RTOL_PREFILL, run_case

SCALE = float(np.float32(1 / math.sqrt(128)))


@pytest.mark.parametrize("B,H,kk,Tq,q_start", [
    (1, 4, 2, 127, 0), (1, 4, 2, 128, 1), (1, 4, 2, 129, 63), (1, 4, 2, 33, 31), (1, 4, 2, 32, 32),   # one, two 128-row tiles
    (2, 6, 3, 385, 64),                                    # four of them, the last with one row
    (66, 4, 2, 70, 5),                                     # more batch rows than one wave adds up at a time
    (40, 32, 8, 65, 130), (40, 16, 4, 129, 100),           # many rows of a short block: 128-row tiles, 256-row tiles
    (14, 32, 8, 257, 3), (14, 32, 8, 512, 0),              # 672: two tiles per group, pairs and singles
    (66, 4, 2, 769, 5),                                    # wide, four tiles, 66 rows
    (5, 24, 24, 1000, 30),                                 # wide, every head alone
    (20, 16, 4, 300, 128), (20, 16, 4, 300, 129), (20, 16, 4, 513, 40),      # three narrow tiles, two wide ones, five narrow
    (26, 16, 4, 700, 5),                                   # 936 wide tiles: six narrow ones
])
def test_prefill_tile_edges(B, H, kk, Tq, q_start):
    print(f"[prefill] B={B} H={H} k={kk} Tq={Tq} q_start={q_start}", flush=True)
    run_case(B, H, kk, Tq, q_start, q_start + Tq + 3, seed=B + 5 * H + 7 * kk + Tq + q_start)


@pytest.mark.parametrize("B,H,Tq,q_start", [(2, 8, 130, 10), (13, 16, 800, 5), (5, 52, 257, 0),
                                            (1, 137, 256, 0), (1, 138, 256, 0), (9, 32, 128, 3),
                                            (30, 20, 1, 0), (2, 8, 64, 0), (2, 8, 64, 1), (30, 20, 128, 0), (2, 8, 33, 95),
                                            (2, 8, 1, 127), (2, 8, 1, 128)])
def test_dense_prefill_tiles(B, H, Tq, q_start):
    """Dense entry point: 128-row tiles; 256-row tiles of eight waves; rings of two up to 128 keys (one tile, two, three)."""
    g = np.random.default_rng(B)
    T = q_start + Tq
    q, k, v = (W.normal(g, (B, H, n, 128), W.BF16) for n in (Tq, T, T))
    out = torch.full((B, H, Tq, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty((C.chai_prefill_workspace_bytes(B, H, H, T),), dtype=torch.uint8, device="cuda")
    C.chai_dense_prefill_attention(dev(q), dev(k), dev(v), q_start, SCALE, out, ws)
    torch.cuda.synchronize()
    ident = np.tile(np.arange(H, dtype=np.int32), (B, 1))
    ok, worst = G.rows_close(out.cpu().numpy(), O.clustered_prefill(q, k, v, ident, ident, q_start, SCALE), RTOL_PREFILL)
    assert ok, worst


@pytest.mark.parametrize("B,Tq", [(1, 200), (24, 300)])
def test_prefill_moving_maximum_and_unused_slot(B, Tq):
    """Keys that grow with their position move the running maximum in block after block (the accumulators are rescaled);
    one slot of the first row is unused and its heads' rows stay untouched."""
    H, kk, q_start = 24, 5, 40
    T = q_start + Tq
    g = np.random.default_rng(Tq)
    q, v = W.normal(g, (B, H, Tq, 128), W.BF16), W.normal(g, (B, H, T, 128), W.BF16)
    k = W.store(g.standard_normal((B, H, T, 128), dtype=np.float32) * (1 + np.arange(T, dtype=np.float32) / 8)[:, None], W.BF16)
    h2c, rep = W.random_membership(g, B, H, kk)
    kc = torch.zeros((B, kk, T, 128), dtype=torch.bfloat16, device="cuda")
    C.chai_compact_kcache(dev(k), dev(rep), kc, T)
    ref = O.clustered_prefill(q, k, v, h2c, rep, q_start, SCALE)
    used = rep.copy()
    used[0, kk - 1] = -1
    out = torch.full((B, H, Tq, 128), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.full((C.chai_prefill_workspace_bytes(B, H, kk, T),), 0xFF, dtype=torch.uint8, device="cuda")
    C.chai_prefill_attention(dev(q), kc, dev(v), dev(h2c), dev(used), q_start, SCALE, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    dead = h2c[0] == kk - 1
    assert dead.any() and np.all(got[0][dead] == 7.0)
    got[0][dead] = ref[0][dead]
    # one key dominates a row here: its probability, 1 before the last rescaling, is exact in fp16; the others carry 2^-11
    ok, worst = G.rows_close(got, ref, RTOL_PREFILL)
    assert ok, worst


def _one_infinite_value(B, H, kk, Tq, q_start, pos):
    """Output of a call whose value cache holds +inf in column 7 at position `pos` of every head, and the oracle's output with
    0 in its place.  kk = 0: the dense entry point."""
    g = np.random.default_rng(B + H + Tq + pos)
    T = q_start + Tq
    q, k, v = (W.normal(g, (B, H, n, 128), W.BF16) for n in (Tq, T, T))
    h2c, rep = W.random_membership(g, B, H, kk) if kk else 2 * (np.tile(np.arange(H, dtype=np.int32), (B, 1)),)
    v[:, :, pos, 7] = 0
    ref = O.clustered_prefill(q, k, v, h2c, rep, q_start, SCALE)
    vd = dev(v)
    vd[:, :, pos, 7] = float("inf")
    out = torch.full((B, H, Tq, 128), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.full((C.chai_prefill_workspace_bytes(B, H, kk or H, T),), 0xFF, dtype=torch.uint8, device="cuda")
    if kk:
        kc = torch.zeros((B, kk, T, 128), dtype=torch.bfloat16, device="cuda")
        C.chai_compact_kcache(dev(k), dev(rep), kc, T)
        C.chai_prefill_attention(dev(q), kc, vd, dev(h2c), dev(rep), q_start, SCALE, out, ws)
    else:
        C.chai_dense_prefill_attention(dev(q), dev(k), vd, q_start, SCALE, out, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy(), ref


@pytest.mark.parametrize("B,H,kk,Tq", [(1, 4, 2, 129), (40, 16, 4, 129), (2, 4, 0, 129), (9, 32, 0, 129), (2, 4, 0, 100)])
def test_infinite_value_reaches_the_rows_that_see_it(B, H, kk, Tq):
    """Narrow and wide tiles, dense narrow and wide ones and rings of two."""
    got, _ = _one_infinite_value(B, H, kk, Tq, 0, 5)
    assert np.all(got[:, :, 5:, 7] == np.inf)


@pytest.mark.parametrize("q_start,pos", [(0, 40), (20, 70), (0, 101)])
@pytest.mark.parametrize("B,H,kk", [(1, 4, 2), (40, 16, 4), (9, 32, 0)])
def test_infinite_value_stays_out_of_blocks_before_it(B, H, kk, q_start, pos):
    """Rows whose block of 32 ends before the value's block of 32 keys begins do not meet it."""
    got, ref = _one_infinite_value(B, H, kk, 140, q_start, pos)
    last = 32 * ((pos // 32 * 32 - 1 - q_start + 1) // 32)        # rows of whole blocks that end before the value's block
    assert last >= 32
    ok, worst = G.rows_close(got[:, :, :last], ref[:, :, :last], RTOL_PREFILL)
    assert ok, worst
    assert np.all(got[:, :, max(pos - q_start, 0):, 7] == np.inf)
