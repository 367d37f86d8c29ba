"""GPU parity of prompt attention where workgroups draw query tile after query tile, at the edges of the queue: every place of the
tickets in the workspace, odd numbers of query tiles, one tile per head, more rows than a wave has lanes, tiles of one and of two
members in turn; against the oracle, and called twice on one workspace."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
from test_gpu_prefill import run_case
from test_gpu_prefill_direct import test_dense_prefill_either_way as dense_case


@pytest.mark.parametrize("B,H,kk,Tq,q_start", [
    (1, 300, 40, 600, 3), (1, 300, 150, 520, 0),           # one row: tickets behind its count; most groups of one member
    (2, 300, 20, 300, 0), (3, 260, 3, 500, 100),           # the last records of two rows; three narrow tiles; two wide ones
    (70, 257, 2, 40, 1),                                   # one query tile per group; more than 64 rows
])
def test_clustered_tiles_are_drawn(B, H, kk, Tq, q_start):
    print(f"[prefill] B={B} H={H} k={kk} Tq={Tq} q_start={q_start}", flush=True)
    run_case(B, H, kk, Tq, q_start, q_start + Tq + 3, seed=B + 5 * H + 7 * kk + Tq + q_start)


@pytest.mark.parametrize("B,H,Tq,q_start", [(3, 200, 700, 130), (9, 70, 300, 258), (2, 300, 512, 200)])
def test_dense_tiles_are_drawn(B, H, Tq, q_start):
    dense_case(B, H, Tq, q_start)


def test_tickets_start_anew_with_every_call():
    """The same workspace, other sizes in between: whatever the last call left in it."""
    torch.manual_seed(3)
    outs = []
    big = C.chai_prefill_workspace_bytes(4, 300, 20, 700)
    ws = torch.full((big,), 0xFF, dtype=torch.uint8, device="cuda")
    data = {}
    for B, Tq in ((4, 700), (1, 600), (4, 700), (2, 512), (4, 700)):
        if (B, Tq) not in data:
            rep = torch.arange(20, dtype=torch.int32).repeat(B, 1)
            h2c = torch.cat([torch.arange(20), torch.randint(0, 20, (280,))]).int().repeat(B, 1)
            data[B, Tq] = (torch.randn(B, 300, Tq, 128).bfloat16().cuda(), torch.randn(B, 20, Tq, 128).bfloat16().cuda(),
                           torch.randn(B, 300, Tq, 128).bfloat16().cuda(), h2c.cuda(), rep.cuda())
        q, k, v, h2c, rep = data[B, Tq]
        out = torch.full((B, 300, Tq, 128), float("nan"), device="cuda")
        C.chai_prefill_attention(q, k, v, h2c, rep, 0, 0.0884, out, ws)
        outs.append(out)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[0], outs[4])
    assert not any(torch.isnan(o).any() for o in outs)
