"""chai_quantize_rows at the edges of its workgroups, codes and scales bit for bit against torch's own cast to 8-bit floats."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2403_08058_amd as C
import workloads as W
from oracle import chai_oracle as O


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


def _want(x):
    """Codes and scales of fp32 rows by the rule, from the table of the 127 finite values: the nearest, of two the even code.  Maxima and
    clamps pass a NaN by: in a row it becomes -448."""
    value = np.array([O.e4m3_decode(c) for c in range(127)])
    with np.errstate(all="ignore"):
        amax = np.fmax.reduce(np.fmax(np.abs(x), np.float32(0)), axis=-1, keepdims=True).astype(np.float32)
        y = np.fmin(np.fmax(x * (np.float32(448) / amax), np.float32(-448)), np.float32(448)).astype(np.float32)
    above = np.clip(np.searchsorted(value, np.abs(y).astype(np.float64)), 1, 126)
    up, down = value[above] - np.abs(y), np.abs(y) - value[above - 1]          # exact in fp64
    code = np.where((up < down) | ((up == down) & (above % 2 == 0)), above, above - 1).astype(np.uint8)
    code = np.where(np.signbit(y), code | 0x80, code).astype(np.uint8)
    code[amax[:, 0] == 0] = 0
    return code, (amax / np.float32(448))[:, 0]


def _check(x, dtype):
    rows = W.bf16_bits_to_f32(W.store(x, W.BF16)) if dtype == torch.bfloat16 else x
    codes, scales = C.chai_quantize_rows(torch.from_numpy(np.ascontiguousarray(rows)).to(dtype).cuda())
    torch.cuda.synchronize()
    code, scale = _want(rows)
    assert np.array_equal(codes.cpu().numpy(), code)
    assert np.array_equal(scales.cpu().numpy(), scale)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_every_code_and_what_lies_halfway(dtype):
    """Rows whose largest element is 448, so that the others are converted as they are: the values of all codes, the middles between
    neighbours and the fp32 (bf16) numbers on either side of both, down to the subnormal codes and what rounds to 0; both signs."""
    value = np.array([O.e4m3_decode(c) for c in range(127)])
    at = np.concatenate([value, (value[1:] + value[:-1]) / 2]).astype(np.float32)
    step = np.float32(2.0 ** -7 if dtype == torch.bfloat16 else 2.0 ** -23)
    all_of_them = np.concatenate([at, at * (1 + step), at * (1 - step), np.float32([1e-30, 1e-40, 2.0 ** -11, 2.0 ** -10])])
    all_of_them = np.concatenate([all_of_them, -all_of_them])
    all_of_them = all_of_them[np.abs(all_of_them) <= 448]
    x = np.zeros((-(-len(all_of_them) // 127), 128), np.float32)
    x[:, 1:].flat[:len(all_of_them)] = all_of_them
    x[:, 0] = 448.0
    _check(x, dtype)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_with_infinities_and_nans(dtype):
    g = np.random.default_rng(3)
    x = g.standard_normal((9, 128)).astype(np.float32)
    x[0, 7], x[1, 9], x[2, 11], x[3, 3] = np.inf, -np.inf, np.nan, -0.0
    x[4, ::3] = np.nan
    x[5] = np.nan                                            # no number at all: as an all-zero row
    x[6, 0], x[6, 1] = np.inf, np.nan
    x[7] *= np.float32(1e-42)                                # 448 over the largest is infinite
    x[7, 5] = 0.0
    _check(x, dtype)
