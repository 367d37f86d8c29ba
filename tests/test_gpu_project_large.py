"""GPU parity of the projection kernel for prompts where a workgroup takes several tiles one after the other: few stages per
tile, ragged tiles, unused slots between used ones.  Reference: the products in 64 bits, with test_gpu_project's bar."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W

import gpu_util as G
from test_gpu_project import check_rounded


@pytest.mark.parametrize("B,H,kk,Tn,D,unused", [
    (16, 24, 20, 100, 64, 0.3),        # one stage per tile: 320 tiles, a workgroup each
    (16, 24, 20, 100, 128, 0.3),       # two stages: 320 tiles on 256 workgroups
    (9, 16, 16, 257, 192, 0.0),        # 288 tiles, every second one of a single token
    (40, 20, 16, 300, 128, 0.9),       # 1280 tiles, most of them of unused slots: workgroups without any
    (11, 12, 12, 512, 320, 0.1),       # 264 whole tiles
])
def test_projection_of_several_tiles_per_workgroup(B, H, kk, Tn, D, unused):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D} unused={unused}", flush=True)
    pos0, cap = 3, Tn + 9
    g = np.random.default_rng(B + Tn + D)
    rep = np.stack([g.permutation(H)[:kk] for _ in range(B)]).astype(np.int32)
    rep[g.random(rep.shape) < unused] = -1
    x, w_q, w_k = (torch.randn(s, generator=torch.Generator("cuda").manual_seed(i), device="cuda").to(torch.bfloat16)
                   for i, s in enumerate([(B, Tn, D), (H * 128, D), (H * 128, D)]))
    q_whole, q_out = G.guarded((B, H, Tn, 128), torch.bfloat16, 3.0)
    k_whole, kc = G.guarded((B, kk, cap, 128), torch.bfloat16, 5.0)
    q_out.fill_(7.0)
    kc.fill_(9.0)
    C.chai_project_qk(x, w_q, w_k, torch.from_numpy(rep).cuda(), q_out, kc, pos0)
    torch.cuda.synchronize()
    assert G.guards_intact(q_whole, (B, H, Tn, 128), 3.0) and G.guards_intact(k_whole, (B, kk, cap, 128), 5.0)
    xs, wq, wk = x.cpu().double(), w_q.cpu().double().view(H, 128, D), w_k.cpu().double().view(H, 128, D)
    qh, kh = W.torch_to_host_bits(q_out), W.torch_to_host_bits(kc)
    nine = W.store(np.array([9.0], np.float32), W.BF16)[0]
    for b in range(B):
        for h in set(range(H)) - set(rep[b].tolist()):
            assert bool((q_out[b, h] == 7.0).all()), "query rows of a pruned head touched"
        for j in range(kk):
            r = int(rep[b, j])
            if r < 0:
                assert np.all(kh[b, j] == nine), "unused slot touched"
                continue
            assert np.all(kh[b, j, :pos0] == nine) and np.all(kh[b, j, pos0 + Tn:] == nine), "rows outside the block touched"
            for got, w, what in ((qh[b, r], wq[r], "q"), (kh[b, j, pos0:pos0 + Tn], wk[r], "k")):
                check_rounded(got, (xs[b] @ w.t()).numpy(), (xs[b].abs() @ w.abs().t()).numpy(), f"{what} b={b} j={j}")


def test_unused_slots_cost_next_to_nothing():
    """8 slots in use of 8 and of 32 (as many as an XCD has workgroups, so that a workgroup that went by slot numbers would meet
    one slot only): the same rows, in much the same time."""
    B, H, Tn, D = 16, 32, 2043, 1024
    rep8 = torch.stack([torch.randperm(H, generator=torch.Generator().manual_seed(b))[:8] for b in range(B)]).int()
    x, w_q, w_k = (torch.randn(s, generator=torch.Generator("cuda").manual_seed(i), device="cuda").to(torch.bfloat16)
                   for i, s in enumerate([(B, Tn, D), (H * 128, D), (H * 128, D)]))
    took, got = {}, {}
    for kk in (8, 32):
        rep = torch.full((B, kk), -1, dtype=torch.int32)
        rep[:, :8] = rep8
        rep = rep.cuda()
        q_out = torch.zeros((B, H, Tn, 128), dtype=torch.bfloat16, device="cuda")
        kc = torch.zeros((B, kk, Tn, 128), dtype=torch.bfloat16, device="cuda")
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            C.chai_project_qk(x, w_q, w_k, rep, q_out, kc, 0)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[kk], got[kk] = sorted(times)[2], (q_out, kc)
    assert torch.equal(got[8][0], got[32][0]) and torch.equal(got[8][1], got[32][1][:, :8]) and not bool(got[32][1][:, 8:].any())
    assert took[32] < 1.8 * took[8], took                    # 3.3 times with workgroups that stand idle
