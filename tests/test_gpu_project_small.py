"""GPU parity of the projection kernels for few tokens (one MFMA row of weights per workgroup; 64-token head-major
tiles) at the edges of their ranges, against the CPU oracle with test_gpu_project's bar (a bf16 neighbour of the exact
value)."""
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
    (8, 32, 8, 1, 256), (1, 32, 8, 8, 64), (1, 5, 5, 7, 576),         # at most eight tokens: weight rows, 4 / 1 / 9 blocks
    (9, 32, 8, 1, 256), (16, 32, 8, 1, 4096),                          # one token more; a decode step of a full batch
    (1, 4, 3, 63, 64), (1, 4, 3, 64, 128), (1, 4, 3, 65, 192),         # around one tile; 1, 2, 3 stages for two teams
    (3, 8, 2, 43, 448),                                                # a tile that gathers tokens of several rows
    (2, 40, 32, 64, 128), (2, 40, 33, 64, 128),                        # 64 tiles (narrow columns), 66 tiles (wide)
    (6, 16, 8, 512, 64), (6, 16, 8, 513, 64),                          # 24576 tokens and more: large tiles
    (2, 257, 3, 20, 64), (1, 256, 3, 20, 64),                          # more heads than a workgroup counts; the most
    (129, 8, 8, 1, 64), (128, 8, 8, 1, 64), (1025, 2, 1, 1, 64),       # more pairs than a workgroup lists; the most
])
def test_projection_of_few_tokens(B, H, kk, Tn, D):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D}", flush=True)
    run_case(B, H, kk, Tn, D, 3, Tn + 7, seed=B * 5 + H * 3 + Tn + D, holes=True)


@pytest.mark.parametrize("Tn", [2, 20])
def test_projection_of_few_tokens_repeated_representative(Tn):
    """One head in two slots of a row: both cache rows are written (weight-row kernel, tile kernel)."""
    B, H, kk, D = 2, 6, 3, 192
    g = np.random.default_rng(Tn)
    x, w_q, w_k = W.normal(g, (B, Tn, D), W.BF16), W.normal(g, (H * 128, D), W.BF16), W.normal(g, (H * 128, D), W.BF16)
    rep = np.array([[4, 1, 4], [5, 4, 0]], np.int32)
    q_out = torch.zeros((B, H, Tn, 128), dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros((B, kk, Tn, 128), dtype=torch.bfloat16, device="cuda")
    C.chai_project_qk(dev(x), dev(w_q), dev(w_k), dev(rep), q_out, kc, 0)
    torch.cuda.synchronize()
    q_ref, k_ref = O.project_qk(x, w_q, w_k, rep, 128)
    x64 = np.abs(W.as_f64(x))
    aq, ak = np.abs(W.as_f64(w_q)).reshape(H, 128, D), np.abs(W.as_f64(w_k)).reshape(H, 128, D)
    qh, kh = W.torch_to_host_bits(q_out), W.torch_to_host_bits(kc)
    for b in range(B):
        for j in range(kk):
            r = int(rep[b, j])
            check_rounded(qh[b, r], q_ref[b, j], np.einsum("te,ce->tc", x64[b], aq[r]), f"q b={b} j={j}")
            check_rounded(kh[b, j], k_ref[b, j], np.einsum("te,ce->tc", x64[b], ak[r]), f"k b={b} j={j}")


@pytest.mark.parametrize("B,H,kk,Tn,D", [
    (4, 8, 8, 512, 192), (4, 8, 8, 513, 192),                          # narrow products: small tiles up to 16384 tokens
    (33, 8, 8, 63, 128),                                               # 264 tiles of 256 tokens: small ones beyond that
])
def test_projection_at_the_lines_of_the_third_round(B, H, kk, Tn, D):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D}", flush=True)
    run_case(B, H, kk, Tn, D, 0, Tn, seed=B + Tn + D, holes=True)
