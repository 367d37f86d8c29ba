"""GPU parity of the projection kernel that streams the weights for a few tokens per head, at the edges of its parts, passes and
look-ups, against the CPU oracle with test_gpu_project's bar (a bf16 neighbour of the exact value)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from test_gpu_project import run_case


@pytest.mark.parametrize("B,H,kk,Tn,D", [
    (1, 32, 8, 1, 64), (1, 32, 9, 1, 128), (1, 40, 17, 1, 512),        # 8 heads in use: one unit each; 9, 17: two; 1, 2, 8 blocks
    (1, 40, 24, 1, 576), (1, 32, 32, 1, 1088),                         # three units, the last part of two; four; 9, 17 blocks
    (1, 52, 40, 2, 192), (1, 64, 51, 1, 704), (1, 80, 64, 1, 256),     # more heads than whole rounds of four units: up to eight
    (1, 90, 72, 1, 320), (2, 300, 150, 1, 128),                        # two rounds; several, five windows of 64 heads
    (1, 4, 3, 8, 192), (1, 4, 3, 9, 192), (1, 4, 3, 16, 192), (1, 4, 3, 17, 192),    # 8, 16 and 32 tokens at a time
    (1, 4, 3, 32, 128), (1, 4, 3, 33, 128), (2, 4, 3, 32, 128),        # one pass and two
    (1, 40, 40, 17, 128),                                              # 32 tokens at a time with six units
    (5, 8, 8, 7, 128), (3, 6, 6, 21, 64),                              # passes that begin inside a row's tokens
    (16, 40, 12, 2, 128), (16, 40, 13, 1, 128),                        # either side of the line to the 64-token tiles
    (1, 40, 8, 64, 64), (8, 40, 9, 5, 64), (17, 33, 33, 3, 64),        # the same for more than 32 tokens
    (64, 20, 17, 1, 64), (64, 4, 4, 1, 64),                            # more pairs than the 64-token tiles list
    (1, 4200, 3, 2, 64),                                               # more heads than a wave's lanes have windows for
])
def test_projection_by_streamed_weights(B, H, kk, Tn, D):
    print(f"[project] B={B} H={H} k={kk} tokens={Tn} width={D}", flush=True)
    run_case(B, H, kk, Tn, D, 3, Tn + 7, seed=B * 5 + H * 3 + Tn + D, holes=B > 1 or kk > 4)
