"""chai_quantize_rows at the edges of its workgroups, codes and scales bit for bit against torch's own cast to 8-bit floats."""
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n_rows", [1, 15, 16, 17, 63, 64, 65, 129, 1000])
def test_rows_are_quantised_whatever_their_number(n_rows, dtype):
    g = torch.Generator().manual_seed(n_rows)
    x = torch.randn((n_rows, 128), generator=g) * torch.exp2(torch.randint(-30, 30, (n_rows, 1), generator=g).float())
    x *= torch.exp2(torch.randint(-18, 1, (n_rows, 128), generator=g).float())       # codes down to the subnormal ones and 0
    x[n_rows // 2] = 0.0
    x[:, 5] = -0.0
    x = x.to(dtype)
    whole = torch.full((n_rows + 2, 128), 0xAA, dtype=torch.uint8, device="cuda")     # guard rows on either side
    sc = torch.full((n_rows + 2,), -7.0, device="cuda")
    codes, scales = C.chai_quantize_rows(x.cuda(), whole[1:-1], sc[1:-1])
    torch.cuda.synchronize()
    amax = x.float().abs().amax(-1, keepdim=True)
    y = (x.float() * torch.where(amax > 0, torch.tensor(448.0) / amax, torch.tensor(0.0))).clamp(-448.0, 448.0)
    want = y.to(torch.float8_e4m3fn).view(torch.uint8)
    want[amax[:, 0] == 0] = 0
    assert torch.equal(codes.cpu(), want)
    assert torch.equal(scales.cpu(), (amax / 448.0)[:, 0])
    assert torch.all(whole[0] == 0xAA) and torch.all(whole[-1] == 0xAA) and sc[0] == -7.0 and sc[-1] == -7.0
