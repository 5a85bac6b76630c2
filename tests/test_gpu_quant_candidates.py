"""slim_quant_search with its candidates in one launch: numbers of bins that are odd, that are no multiple of a workgroup's
1024 or of its ten counts in flight, and the largest; calls in turn on one workspace, whose counts of ended
workgroups and errors are left over from the call before.  alpha* is the oracle's (or a candidate of equal error)."""
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
