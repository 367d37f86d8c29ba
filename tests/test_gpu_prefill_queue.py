"""GPU parity of prompt attention where workgroups draw query tile after query tile, at the edges of the queue: every place of the
tickets in the workspace, odd numbers of query tiles, one tile per head, more rows than a wave has lanes, tiles of one and of two
members in turn; against the oracle, and called twice on one workspace."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
from test_gpu_prefill import RTOL_PREFILL, run_case
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


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("Tq,q_start", [(16128, 3), (16129, 0)])
def test_prompts_of_thirty_two_pairs_of_tiles(Tq, q_start, dense):
    """Long prompts' pairs stand in the queue by the round, odd and even numbers of tiles: the same rows as in blocks of a few tiles, whose
    pairs stand there one by one.  Both round the probabilities to 11 bits and add in 32: each is within test_gpu_prefill's bound of the
    exact row, and so within twice that of the other."""
    B, H, kk, n = 1, 40, 8, q_start + Tq
    g = torch.Generator(device="cuda").manual_seed(Tq)
    normal = lambda *shape: torch.randn(shape, generator=g, device="cuda").bfloat16()  # noqa: E731
    q, k, v = normal(B, H, Tq, 128), normal(B, H if dense else kk, n, 128), normal(B, H, n, 128)
    rep = torch.arange(kk, dtype=torch.int32).repeat(B, 1).cuda()
    h2c = torch.cat([torch.arange(kk), torch.arange(H - kk) % kk]).int().repeat(B, 1).cuda()
    ws = torch.zeros(C.chai_prefill_workspace_bytes(B, H, H if dense else kk, n), dtype=torch.uint8, device="cuda")

    def attention(qs, start, out):
        if dense:
            C.chai_dense_prefill_attention(qs, k, v, start, 0.0884, out, ws)
        else:
            C.chai_prefill_attention(qs, k, v, h2c, rep, start, 0.0884, out, ws)

    whole = torch.full((B, H, Tq, 128), float("nan"), device="cuda")
    attention(q, q_start, whole)
    for i in range(0, Tq, 4096):
        rows = q[:, :, i:i + 4096].contiguous()
        part = torch.full((B, H, rows.shape[2], 128), float("nan"), device="cuda")
        attention(rows, q_start + i, part)
        err = (whole[:, :, i:i + 4096] - part).abs().amax(dim=-1) / part.abs().amax(dim=-1)
        assert err.max() <= 2 * RTOL_PREFILL             # (false for a NaN)
