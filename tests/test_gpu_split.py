"""The products of the adapter computation on two fp16 numbers per operand (csrc/slim_lora_split.hip) by themselves, element by element
against binary64, with operands whose rows, channels and block entries lie far below the largest ones.  The bound of an element is
relative to the sum of the magnitudes of its products: 2^-22 each for the two numbers of either operand and for the product of the
second ones that is left out, and a rounding of binary32 for each of K / 16 + 16 partial sums."""
import ctypes

import pytest
import torch

from paper_2410_09615_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SPLIT, LOW = 64.0, 2048.0            # scale of a block, of a second number


def _halves(count):
    return torch.empty(count, dtype=torch.half, device=DEV)


def _products(S, Z, Q):
    """(S Z, S^T Q) by the library."""
    n, k = S.shape
    n32, l = -(-n // 32) * 32, Z.shape[1]
    vp, i32 = ctypes.c_void_p, ctypes.c_int
    split, gemm, shares = (getattr(B.lib(), "_ZN4slim" + s) for s in (
        "17launch_lora_splitEPKfiiPKjS3_PDF16_S4_S4_S4_PfP12ihipStream_t",
        "22launch_lora_split_gemmEPKDF16_S1_PKjPKfS1_S1_iiiPfS6_PjP12ihipStream_t", "17split_gemm_splitsEiii"))
    split.argtypes = [vp, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    gemm.argtypes = [vp, vp, vp, vp, vp, vp, i32, i32, i32, vp, vp, vp, vp]
    st = torch.cuda.current_stream().cuda_stream
    largest, channels, factor = S.abs().amax(), torch.zeros(8, k, device=DEV), torch.empty(k, device=DEV)
    channels[2], channels[7, ::2] = 0.4 * S.abs().amax(0), S.abs().amax(0)[::2]       # (the largest of the eight rows counts)
    channels[5, 1::2] = S.abs().amax(0)[1::2]
    half = [_halves(n32 * k) for _ in range(4)]
    assert split(S.data_ptr(), n, k, largest.data_ptr(), channels.data_ptr(), *[h.data_ptr() for h in half], factor.data_ptr(), st) == 0

    def pair(A, rows):               # columns as rows
        v = torch.zeros(l, rows, device=DEV)
        v[:, :A.shape[0]] = A.T * SPLIT
        hi = v.half()
        return hi, ((v - hi.float()) * LOW).half()

    out = []
    for A, at, rows, cols, scale, factors in ((Z, 0, n, k, largest, None), (Q, 2, k, n32, None, factor)):
        hi, lo = pair(A, cols)
        P, Y = torch.empty(shares(rows, l, cols) * rows * l, device=DEV), torch.empty(rows, l, device=DEV)
        assert gemm(half[at].data_ptr(), half[at + 1].data_ptr(), None if scale is None else scale.data_ptr(),
                    None if factors is None else factors.data_ptr(), hi.data_ptr(), lo.data_ptr(), rows, l, cols, P.data_ptr(), Y.data_ptr(), None, st) == 0
        out.append(Y)
    torch.cuda.synchronize()
    return out


def _check(S, Z, Q):
    for got, A, V in zip(_products(S, Z, Q), (S.double(), S.double().T), (Z.double(), Q.double())):
        size = A.abs() @ V.abs()
        bound = (3 * 2.0 ** -22 + (A.shape[1] / 16 + 16) * 2.0 ** -24) * size
        assert bool(((got.double() - A @ V).abs() <= bound + 2.0 ** -126).all())


def _gauss(*shape, seed):
    return torch.randn(*shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV)


@pytest.mark.parametrize("n,k,l", [(70, 128, 32), (513, 640, 96), (1000, 1152, 416)])
@pytest.mark.parametrize("kind", ["even", "rows", "block", "channels"])
def test_products_of_two_fp16_numbers(n, k, l, kind):
    """rows: half of the rows of W 2^26 below the others, and a block that is zero on those, as directions are that only small rows have.
    block: entries 2^13 below the largest of the block, which meet zeros of S.  channels: magnitudes over 2^60 (and one of zeros), whatever the
    saliency is."""
    S, Z, Q = _gauss(n, k, seed=1), _gauss(k, l, seed=2) * k ** -0.5, _gauss(n, l, seed=3) * n ** -0.5
    if kind == "rows":
        S[::2] *= 2.0 ** -26
        Q[1::2] = 0
    if kind == "block":
        Q[::2] *= 2.0 ** -13
        Z[::2] *= 2.0 ** -13
        S[1::2] = 0
        S[:, 1::2] = 0
    if kind == "channels":
        S *= torch.exp2(torch.linspace(-30, 30, k, device=DEV)[torch.randperm(k, generator=torch.Generator().manual_seed(5))])
        S[:, 7] = 0
    _check(S, Z, Q)
