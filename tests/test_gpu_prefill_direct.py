"""GPU parity of the prefill kernel that converts the values itself (few query tiles per head) at the edges of its tiles and of
the sizes it takes, and of the kernels behind the pre-pass at sizes that one would take with fewer heads."""
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
from test_gpu_prefill_tiles import SCALE, _one_infinite_value


@pytest.mark.parametrize("B,H,kk,Tq,q_start", [
    (1, 2, 1, 1, 0), (1, 1, 1, 31, 0), (3, 5, 2, 64, 0), (3, 5, 2, 65, 0), (1, 7, 3, 3, 61), (1, 7, 3, 3, 62),   # 1, 2 key tiles
    (1, 3, 1, 1, 127), (1, 3, 1, 1, 128), (2, 3, 1, 5, 187), (2, 3, 1, 5, 188), (1, 6, 2, 100, 477),             # 2 .. 10 of them
    (5, 64, 9, 20, 50), (3, 65, 64, 40, 30), (1, 256, 64, 33, 10), (2, 200, 3, 40, 5),                           # heads, clusters
    (9, 70, 11, 250, 6),                                   # several rounds of workgroups
    (1, 6, 2, 897, 0), (1, 16, 3, 1024, 5),                # eight query tiles
])
def test_prefill_direct_edges(B, H, kk, Tq, q_start):
    print(f"[prefill] B={B} H={H} k={kk} Tq={Tq} q_start={q_start}", flush=True)
    run_case(B, H, kk, Tq, q_start, q_start + Tq + 3, seed=B + 5 * H + 7 * kk + Tq + q_start)


@pytest.mark.parametrize("B,H,kk,Tq,q_start", [
    (1, 257, 3, 40, 5), (1, 70, 65, 40, 5),                # one head, one cluster more than it takes
    (1, 260, 4, 129, 64), (4, 260, 4, 150, 3), (5, 260, 4, 300, 0),              # narrow, wide, three narrow tiles
    (1, 6, 2, 1025, 7), (1, 32, 8, 20, 1600),              # nine query tiles; a long chain of few heads
    (11, 52, 8, 900, 300),                                 # eight tiles of many heads
])
def test_prefill_behind_the_pre_pass(B, H, kk, Tq, q_start):
    print(f"[prefill] B={B} H={H} k={kk} Tq={Tq} q_start={q_start}", flush=True)
    run_case(B, H, kk, Tq, q_start, q_start + Tq + 3, seed=B + 5 * H + 7 * kk + Tq + q_start)


@pytest.mark.parametrize("B,H,Tq,q_start", [
    (2, 8, 64, 1), (1, 1, 1, 0), (1, 5, 17, 180), (70, 5, 130, 3),               # converting values
    (41, 50, 60, 4), (41, 50, 60, 5), (32, 64, 3, 0),      # 2050 heads, one key tile (behind the pre-pass) and two
    (1, 33, 1000, 0), (7, 40, 300, 300), (1, 8, 40, 2500), # eight tiles, second round; three; few heads
    (7, 45, 500, 129),
])
def test_dense_prefill_either_way(B, H, Tq, q_start):
    print(f"[dense prefill] B={B} H={H} Tq={Tq} q_start={q_start}", flush=True)
    g = np.random.default_rng(B + H + Tq)
    T, cap = q_start + Tq, q_start + Tq + 2
    q, k, v = W.normal(g, (B, H, Tq, 128), W.BF16), W.normal(g, (B, H, cap, 128), W.BF16), W.normal(g, (B, H, cap, 128), W.BF16)
    k[:, :, T:], v[:, :, T:] = np.uint16(0x7FC0), np.uint16(0x7FC0)              # positions past the block are never read
    whole, out = G.guarded((B, H, Tq, 128), torch.float32, float("nan"))
    ws = torch.full((C.chai_prefill_workspace_bytes(B, H, H, T),), 0xFF, dtype=torch.uint8, device="cuda")
    C.chai_dense_prefill_attention(dev(q), dev(k), dev(v), q_start, SCALE, out, ws)
    torch.cuda.synchronize()
    ident = np.tile(np.arange(H, dtype=np.int32), (B, 1))
    ok, worst = G.rows_close(out.cpu().numpy(), O.clustered_prefill(q, k, v, ident, ident, q_start, SCALE), RTOL_PREFILL)
    assert ok, worst
    assert G.guards_intact(whole, (B, H, Tq, 128), float("nan"))


@pytest.mark.parametrize("Tq,q_start", [(1, 0), (8, 5), (16, 0), (17, 47), (31, 33), (32, 32), (33, 0), (48, 16), (49, 15), (64, 0), (16, 49), (17, 100)])
def test_short_blocks_of_one_tile_of_keys(Tq, q_start):
    """One tile of keys has a start of its own, and up to 16 rows of a wave half of its stores (the last two: two tiles)."""
    print(f"[prefill] Tq={Tq} q_start={q_start}", flush=True)
    run_case(2, 9, 3, Tq, q_start, q_start + Tq + 3, seed=Tq + q_start)
    test_dense_prefill_either_way(3, 5, Tq, q_start)         # converting values
    test_dense_prefill_either_way(41, 50, Tq, q_start)       # two workgroups per CU, behind the pre-pass


def test_prefill_direct_unassigned_heads_and_unused_slots():
    """Heads without a cluster, or of a cluster without a representative, keep their rows; the others' groups close ranks."""
    B, H, kk, Tq, q_start = 3, 23, 5, 70, 9
    T = q_start + Tq
    g = np.random.default_rng(4)
    q, k, v = (W.normal(g, (B, H, n, 128), W.BF16) for n in (Tq, T, T))
    h2c, rep = W.random_membership(g, B, H, kk)
    kc = torch.zeros((B, kk, T, 128), dtype=torch.bfloat16, device="cuda")
    C.chai_compact_kcache(dev(k), dev(rep), kc, T)
    ref = O.clustered_prefill(q, k, v, h2c, rep, q_start, SCALE)
    h2c, used = h2c.copy(), rep.copy()
    used[0, 0] = used[1, 2] = used[1, 4] = -1
    loose = np.zeros((B, H), bool)
    for b in range(B):
        loose[b] = used[b][h2c[b]] < 0
        for h in np.flatnonzero(~loose[b] & ~np.isin(np.arange(H), rep[b]))[:2]:
            h2c[b, h] = -1 if h % 2 else kk
            loose[b, h] = True
    assert loose.any(1).all() and not loose.all(1).any()
    out = torch.full((B, H, Tq, 128), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.empty((C.chai_prefill_workspace_bytes(B, H, kk, T),), dtype=torch.uint8, device="cuda")
    C.chai_prefill_attention(dev(q), kc, dev(v), dev(h2c), dev(used), q_start, SCALE, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.all(got[loose] == 7.0)
    ok, worst = G.rows_close(got[~loose], ref[~loose], RTOL_PREFILL)
    assert ok, worst


@pytest.mark.parametrize("q_start,pos", [(0, 40), (20, 70), (0, 101)])
@pytest.mark.parametrize("B,H,kk", [(1, 260, 4), (4, 260, 4), (1, 6, 0)])
def test_infinite_value_behind_the_pre_pass_and_direct(B, H, kk, q_start, pos):
    got, ref = _one_infinite_value(B, H, kk, 140, q_start, pos)
    last = 32 * ((pos // 32 * 32 - 1 - q_start + 1) // 32)
    ok, worst = G.rows_close(got[:, :, :last], ref[:, :, :last], RTOL_PREFILL)
    assert last >= 32 and ok, worst
    assert np.all(got[:, :, max(pos - q_start, 0):, 7] == np.inf)
