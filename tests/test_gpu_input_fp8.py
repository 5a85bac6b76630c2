"""The 8-bit codes of the input quantizer over every fp16 value, against the oracle, and what it does with values that are not finite."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2410_09615_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# largest magnitudes: one bit in the last place of a binade's ends, both sides of the change of format, subnormal ones
@pytest.mark.parametrize("M", [65504.0, 449.0, 448.25, 448.0, 447.75, 7.0, 6.996, 5.437, 1.0, 0.9995, 3.1e-3, 6.104e-5, 6.0e-5, 5.960e-8])
def test_every_value_below_a_maximum(M):
    M = float(np.float16(M))
    pos = np.arange(0x7C00, dtype=np.uint16).view(np.float16)
    pos = pos[pos.astype(np.float32) <= M]
    X = np.concatenate([pos, -pos, pos[-1:]])                                  # an odd count: the tail has its own code
    Xq, info, codes = B.slim_input_quant_fp8(torch.from_numpy(X).to(DEV), codes=True)
    _, _, alone = B.slim_input_quant_fp8(torch.from_numpy(X).to(DEV), Xq=False, codes=True)
    torch.cuda.synchronize()
    rc, rs, rf = O.input_quant_fp8_codes(X)
    rq, _, _ = O.input_quant_fp8(X)
    assert float(info[0]) == float(np.float32(rs)) and float(info[1]) == (1.0 if rf == "e5m2" else 0.0)
    assert np.array_equal(codes.cpu().numpy(), rc) and torch.equal(codes, alone)
    assert np.array_equal(Xq.cpu().numpy().view(np.uint16), rq.view(np.uint16))


@pytest.mark.parametrize("count", [1, 7, 8, 9, 2047, 2048, 2049, 8 * 2048 * 256 + 8, 8 * 4096 * 256 + 13])
def test_lengths(count):
    """One and several pieces per lane, with and without a tail."""
    g = torch.Generator().manual_seed(count)
    X = torch.randn(count, generator=g).half()
    _, info, codes = B.slim_input_quant_fp8(X.to(DEV), Xq=False, codes=True)
    torch.cuda.synchronize()
    rc, rs, _ = O.input_quant_fp8_codes(X.numpy())
    assert float(info[0]) == float(np.float32(rs))
    assert np.array_equal(codes.cpu().numpy(), rc)


def test_not_finite():
    """A NaN does not count for the maximum and gets the largest code; with an infinity the scale is infinite, every finite value gets
    code 0 and the infinity the largest code."""
    X = torch.ones(64, dtype=torch.float16)
    X[3] = float("nan")
    X[4] = -0.5
    _, info, codes = B.slim_input_quant_fp8(X.to(DEV), Xq=False, codes=True)
    assert float(info[0]) == float(np.float32(1.0) / np.float32(448.0))
    want = torch.full((64,), 0x7E, dtype=torch.uint8)
    want[4] = 0x80 | 0x76
    assert torch.equal(codes.cpu() & 0x7F, want & 0x7F) and int(codes[4]) == 0xF6
    X[9], X[10] = float("inf"), -float("inf")
    Xq, info, codes = B.slim_input_quant_fp8(X.to(DEV), codes=True)
    assert float(info[0]) == float("inf") and float(info[1]) == 1.0
    want = torch.zeros(64, dtype=torch.uint8)
    want[[3, 9, 10]] = 0x7B
    want[4], want[10] = 0x80, 0xFB
    codes = codes.cpu()
    assert torch.equal(codes & 0x7F, want & 0x7F) and int(codes[4]) == 0x80 and int(codes[10]) == 0xFB
    assert bool(torch.isnan(Xq[0])) and bool(torch.isinf(Xq[9]))
