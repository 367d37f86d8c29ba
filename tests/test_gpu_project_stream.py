"""GPU parity of the projection kernel that streams the weights for a few tokens per head, at the edges of its parts, passes and
look-ups, and of the calls on either side of the lines to the other kernels, against the CPU oracle with test_gpu_project's bar (a bf16
neighbour of the exact value)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W
from oracle import chai_oracle as O

from gpu_util import dev
from test_gpu_project import check_rounded, run_case


@pytest.mark.parametrize("B,H,kk,Tn,D", [
    # (most of the narrow ones go to the other kernels: the same sizes at widths that are streamed stand below)
    (1, 32, 8, 1, 64), (1, 32, 9, 1, 128), (1, 40, 17, 1, 512),        # 17 heads in use: two units each; 8 blocks
    (1, 40, 24, 1, 576), (1, 32, 32, 1, 1088),                         # four units; 9, 17 blocks
    (1, 52, 40, 2, 192), (1, 64, 51, 1, 704), (1, 80, 64, 1, 256),     # more heads than whole rounds of four units: up to eight
    (1, 90, 72, 1, 320), (2, 300, 150, 1, 128),                        # two rounds
    (1, 4, 3, 8, 192), (1, 4, 3, 9, 192), (1, 4, 3, 16, 192), (1, 4, 3, 17, 192),
    (1, 4, 3, 32, 128), (1, 4, 3, 33, 128), (2, 4, 3, 32, 128),
    (1, 40, 40, 17, 128), (5, 8, 8, 7, 128), (3, 6, 6, 21, 64),
    (16, 40, 12, 2, 128), (16, 40, 13, 1, 128), (1, 40, 8, 64, 64), (8, 40, 9, 5, 64), (17, 33, 33, 3, 64),
    (64, 20, 17, 1, 64), (64, 4, 4, 1, 64),                            # more pairs than the 64-token tiles list; a quarter of what they do
    (1, 4200, 3, 2, 64),                                               # more heads than a wave's lanes have windows for
])
def test_projection_by_streamed_weights(B, H, kk, Tn, D):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D}", flush=True)
    run_case(B, H, kk, Tn, D, 3, Tn + 7, seed=B * 5 + H * 3 + Tn + D, holes=B > 1 or kk > 4)


def _repeats(B, H, kk, used, head, copies, past_the_end):
    """Maps with `used` heads in use, `head` in the first copies[b] slots of row b, and a last slot of row 0 that names no head."""
    others = [h for h in range(H) if h != head][:used - 1]
    rep = np.full((B, kk), -1, np.int32)
    at = 0
    for b in range(B):
        rep[b, :copies[b]] = head
        for j in range(copies[b], kk - (1 if past_the_end and b == 0 else 0)):
            if at < len(others):
                rep[b, j] = others[at]
                at += 1
    assert at == len(others)
    if past_the_end:
        rep[0, kk - 1] = H + 3
    return rep


@pytest.mark.parametrize("B,H,kk,Tn,D,used,head,copies,past_the_end", [
    (1, 72, 64, 8, 320, 63, 5, [2], False),                # eight units: 16 tokens of one head are one pass,
    (1, 72, 64, 6, 1088, 62, 5, [3], False),               # 18 two; 3 blocks for the first wave
    (1, 72, 64, 8, 256, 60, 71, [5], False),               # three, each of whole slots
    (1, 80, 80, 1, 576, 64, 0, [17], False),               # 17 slots of one token
    (1, 64, 48, 7, 320, 46, 9, [3], False),                # seven units, passes that begin inside a slot's tokens
    (2, 72, 30, 4, 320, 47, 60, [3, 2], False),            # repeats in two rows: 20 tokens
    (4, 72, 16, 4, 4096, 60, 71, [1, 1, 1, 1], True),      # an entry past the last head, whose tokens the last head gets
    (2, 72, 40, 4, 256, 58, 71, [2, 2], True),
    (2, 52, 20, 4, 512, 32, 3, [3, 3], False),             # at most six units: 24 tokens at once
    (1, 40, 36, 8, 512, 32, 3, [5], False),                # 40 in two passes
])
def test_streamed_projection_of_a_repeated_representative(B, H, kk, Tn, D, used, head, copies, past_the_end):
    """A head that stands in several slots has more tokens than the batch has: every slot's keys and the head's queries are written,
    whatever number of units a workgroup takes."""
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D} used={used} copies={copies}", flush=True)
    g = np.random.default_rng(used + Tn)
    x, w_q, w_k = W.normal(g, (B, Tn, D), W.BF16), W.normal(g, (H * 128, D), W.BF16), W.normal(g, (H * 128, D), W.BF16)
    rep = _repeats(B, H, kk, used, head, copies, past_the_end)
    q_out = torch.zeros((B, H, Tn, 128), dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros((B, kk, Tn, 128), dtype=torch.bfloat16, device="cuda")
    C.chai_project_qk(dev(x), dev(w_q), dev(w_k), dev(rep), q_out, kc, 0)
    torch.cuda.synchronize()
    q_ref, k_ref = O.project_qk(x, w_q, w_k, np.minimum(rep, H - 1), 128)
    x64 = np.abs(W.as_f64(x))
    aq, ak = np.abs(W.as_f64(w_q)).reshape(H, 128, D), np.abs(W.as_f64(w_k)).reshape(H, 128, D)
    qh, kh = W.torch_to_host_bits(q_out), W.torch_to_host_bits(kc)
    for b in range(B):
        for j in range(kk):
            r = int(rep[b, j])
            if 0 <= r < H:
                check_rounded(qh[b, r], q_ref[b, j], np.einsum("te,ce->tc", x64[b], aq[r]), f"q b={b} j={j}")
                check_rounded(kh[b, j], k_ref[b, j], np.einsum("te,ce->tc", x64[b], ak[r]), f"k b={b} j={j}")


@pytest.mark.parametrize("B,H,kk,Tn,D", [
    (1, 32, 8, 1, 640), (1, 32, 8, 8, 576),                           # few heads: one unit each; just too narrow to be streamed
    (1, 32, 9, 1, 384), (1, 32, 9, 3, 320), (1, 40, 17, 1, 576), (1, 40, 23, 1, 512), (1, 52, 40, 2, 512),      # two units; three; six
    (1, 64, 51, 1, 256), (1, 64, 51, 1, 192), (1, 64, 64, 2, 4096), (1, 64, 64, 3, 4096),      # rows on the same memory channels
    (1, 256, 200, 1, 512), (2, 300, 150, 1, 512), (1, 257, 128, 8, 64), (1, 600, 300, 4, 448),                  # several rounds, windows
    (1, 4, 3, 8, 2560), (1, 4, 3, 9, 1024), (1, 4, 3, 16, 1024), (1, 4, 3, 17, 1024),                           # 8, 16, 32 tokens at a time
    (1, 4, 3, 32, 1024), (1, 4, 3, 32, 960), (1, 4, 3, 33, 2048), (2, 4, 3, 32, 2048),                          # one pass and two
    (5, 8, 8, 7, 2048), (3, 6, 6, 21, 2048), (1, 40, 40, 17, 2560),                                             # passes inside a row's tokens
    (16, 40, 12, 2, 2560), (16, 40, 12, 2, 2496), (3, 6, 6, 5, 1024), (3, 6, 6, 5, 960), (1, 40, 8, 64, 2048), (1, 52, 51, 8, 4096), (1, 52, 52, 8, 4096),
    (16, 72, 72, 1, 1088), (4, 300, 2, 4, 128), (2, 400, 200, 16, 576),      # no other kernel but 256-token tiles
    (4, 300, 30, 3, 192), (4, 300, 30, 3, 256), (2, 300, 60, 4, 192), (2, 300, 60, 4, 256), (1, 64, 64, 2, 8192),
])
def test_projection_on_either_side_of_the_lines(B, H, kk, Tn, D):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D}", flush=True)
    run_case(B, H, kk, Tn, D, 3, Tn + 7, seed=B * 5 + H * 3 + Tn + D, holes=B > 1 or kk > 4)
