"""slim_pack and slim_pack_ex on both sides of the row lengths where the kernel changes, and on quotients that lie on a half or next to
one, against the oracle's mask and codes (bit for bit)."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2410_09615_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(W, sal, given):
    n, k = W.shape
    q, m, s = B.slim_pack_ex(torch.from_numpy(W).to(DEV), None if sal is None else torch.from_numpy(sal).to(DEV),
                             None if given is None else torch.from_numpy(given).to(DEV))
    codes, mask = B.slim_unpack(q, m, n, k)
    torch.cuda.synchronize()
    ref_mask = O.mask_2of4(W, sal)
    ref_scale = O.row_scale(W) if given is None else given
    assert np.array_equal(s.cpu().numpy(), ref_scale)
    assert np.array_equal(mask.cpu().numpy(), ref_mask)
    assert np.array_equal(codes.cpu().numpy(), O.quantize(W, ref_mask, ref_scale))


@pytest.mark.parametrize("n,k", [(1, 8), (33, 2048), (31, 2056), (17, 8192), (16, 8200), (15, 16384), (5, 16392), (5, 32768), (3, 32776), (2, 49160)])
def test_row_lengths(n, k):
    rng = np.random.default_rng(k)
    W = rng.standard_normal((n, k)).astype(np.float32)
    W[:, ::5] = np.round(W[:, ::5] * 2) / 2                      # equal magnitudes: the lower position is kept
    sal = rng.uniform(0.1, 3.0, k).astype(np.float32)
    given = rng.uniform(0.05, 0.6, n).astype(np.float32)
    for use_sal in (False, True):
        for use_scale in (False, True):
            check(W, sal if use_sal else None, given if use_scale else None)


@pytest.mark.parametrize("n,k", [(2, 53256), (33, 57352), (1, 65536), (2, 36864)])
def test_row_lengths_that_are_read_twice(n, k):
    """Four groups per lane at a time, from the end: every remainder of the number of trips."""
    rng = np.random.default_rng(k + 1)
    W = rng.standard_normal((n, k)).astype(np.float32)
    check(W, None, None)
    check(W, rng.uniform(0.1, 3.0, k).astype(np.float32), None)


@pytest.mark.parametrize("scale", [0.5, 0.1, 1 / 7.0, 3.3333333, 1e-30, 1e-40, 1e36])
def test_quotients_next_to_a_half(scale):
    """Products of the scale with every half from -9.5 to 8.5, and the four numbers on both sides of each."""
    s = np.float32(scale)
    halves = (np.arange(-9.5, 9.0) * np.float64(s)).astype(np.float32)
    rows = [halves]
    up, down = halves, halves
    for _ in range(4):
        up, down = np.nextafter(up, np.float32(np.inf)), np.nextafter(down, np.float32(-np.inf))
        rows += [up, down]
    flat = np.concatenate(rows)
    W = np.zeros((1, 4 * ((flat.size + 7) // 8 * 8)), np.float32)
    W[0, 1:4 * flat.size:4] = flat                               # one of each group, so that every one is kept
    check(W, None, np.array([s], np.float32))
