"""slim_quant_search with its candidates in one launch: numbers of bins that are odd, that are no multiple of a workgroup's
1024 or of its ten counts in flight, and the largest; calls in turn on one workspace, whose counts of ended
workgroups and errors are left over from the call before.  alpha* is the oracle's (or a candidate of equal error)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2410_09615_amd import binding as B
from paper_2410_09615_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,k", [(1, 8), (513, 1000), (1001, 1024), (1300, 2048), (3001, 3400), (2600, 8192)])
def test_candidates_in_one_launch(n, k):
    W = wl.make_weight(n, k, seed=n).numpy()
    W[0, 0] *= 3.0
    Wd = torch.from_numpy(W).to(DEV)
    for _ in range(2):
        scale, alpha = B.slim_quant_search(Wd)
        torch.cuda.synchronize()
        a = np.float32(alpha.cpu().numpy().reshape(-1)[0])
        assert O.quant_search_accepts(W, a)
        assert np.all(scale.cpu().numpy() == np.float32(a / np.float32(7.0)))


def test_calls_in_turn_on_one_workspace():
    """One workspace for tensors with different alpha* and different numbers of bins (so that what one call counted lies
    where another keeps its errors), filled with 0xFF before the first call: counts of ended workgroups that are not
    cleared, or errors read before they are written, would show as another tensor's alpha*."""
    lib = B.lib()
    tensors = []
    for i, (n, k) in enumerate([(513, 1000), (3001, 3400), (1001, 1024), (2600, 8192), (1, 8)]):
        W = wl.make_weight(n, k, seed=50 + i).numpy() * 4.0 ** i
        W[0, 0] *= 1.0 + i
        tensors.append((W, torch.from_numpy(W).to(DEV), torch.empty(n, dtype=torch.float32, device=DEV), torch.empty(1, dtype=torch.float32, device=DEV)))
    sizes = []
    for W, _, _, _ in tensors:
        b = ctypes.c_size_t()
        assert lib.slim_quant_workspace_bytes(B.slim_shape(*W.shape, 0), b) == 0
        sizes.append(b.value)
    ws = torch.full((max(sizes),), 255, dtype=torch.uint8, device=DEV)
    order = [0, 1, 2, 1, 3, 0, 4, 3, 2, 0, 1]
    for i in order:
        W, Wd, scale, alpha = tensors[i]
        scale.fill_(-1.0)
        alpha.fill_(-1.0)
        assert lib.slim_quant_search(B._ptr(Wd), B.slim_shape(*W.shape, 0), B._ptr(scale), B._ptr(alpha), B._ptr(ws), sizes[i],
                                     B._stream(Wd)) == 0
        torch.cuda.synchronize()
        a = np.float32(alpha.cpu().numpy()[0])
        assert O.quant_search_accepts(W, a)
        assert np.all(scale.cpu().numpy() == np.float32(a / np.float32(7.0)))


@pytest.mark.parametrize("n,k", [(3, 8), (5, 520), (2, 512992), (2, 513000), (2, 520000)])
@pytest.mark.parametrize("dist", ["normal", "student_t", "one_value"])
def test_rows_with_and_without_a_table_of_bins(n, k, dist):
    """Rows of 512 bins, whose centres and counts are tabulated, and of more (from 513000 inputs on); most bins empty, all but one."""
    rng = np.random.default_rng(k)
    if dist == "normal":
        W = rng.standard_normal((n, k)).astype(np.float32) * 0.02
    elif dist == "student_t":
        W = rng.standard_t(2, (n, k)).astype(np.float32)
    else:
        W = np.full((n, k), 0.5, np.float32)
    W[n - 1] *= np.float32(1e-3)
    scale, alpha = B.slim_quant_search_rows(torch.from_numpy(W).to(DEV))
    torch.cuda.synchronize()
    a = alpha.cpu().numpy().reshape(-1)
    for i in range(n):
        assert O.quant_search_accepts(W[i:i + 1], a[i])
    assert np.array_equal(scale.cpu().numpy(), (a / np.float32(7.0)).astype(np.float32))
