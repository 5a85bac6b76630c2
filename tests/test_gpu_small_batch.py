"""slim_linear_gemm, slim_linear_gemm_fp8 and slim_lowrank on batches of 17 to 512 tokens (mid_kernel,
csrc/slim_gemm_mid.hip) against the oracle, at the sizes where that path can go wrong: each of its four tile
shapes with whole, ragged and partly empty tiles, T made in the same launch and in one of its own, one stage of
inputs, stage counts that are no multiple of a round, ranks below and beyond whole rounds of the adapter term.
The bounds are those of parity.py."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import slim_oracle as O
from paper_2410_09615_amd import binding as B
from paper_2410_09615_amd import workloads as wl
from parity import TOL_Y
from test_gpu_parity import (CT_PREFILL, DEV, _assert_layer_close, _assert_lowrank_close, _forward_case, _fp8_forward_case,
                             _gpu_layer, _shape)

pytestmark = pytest.mark.gpu

# tile rows x tokens: 32 x 32, 64 x 32, 128 x 32, 128 x 64 (the smallest that leaves every compute unit at most one)
CASES = [
    (512, 512, 51, 17), (33, 128, 1, 31), (32, 384, 31, 32), (1001, 640, 33, 70), (130, 2176, 97, 129), (700, 4096, 409, 33),
    (4096, 256, 64, 64), (5000, 1408, 96, 40), (2049, 640, 200, 96), (1500, 1152, 150, 200),
    (9001, 384, 65, 48), (11008, 640, 34, 33), (3000, 1280, 300, 160),
    (28000, 256, 90, 40), (20003, 384, 130, 64), (4096, 512, 51, 512), (2050, 1152, 1100, 500),
    (28672, 256, 60, 100), (700, 2048, 0, 40), (9001, 256, 0, 200),
]


@pytest.mark.parametrize("n,k,r,m", CASES)
def test_small_batch(n, k, r, m):
    assert _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=21) <= TOL_Y


@pytest.mark.parametrize("n,k,r,m", [c for c in CASES if c[2] > 0])
def test_small_batch_q4_adapters(n, k, r, m):
    assert _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=22, bits=4) <= TOL_Y


@pytest.mark.parametrize("bits", [16, 4])
@pytest.mark.parametrize("gain", [1.0, 300.0])
@pytest.mark.parametrize("n,k,r,m", [CASES[i] for i in (1, 3, 5, 7, 9, 10, 12, 13, 16, 17)])
def test_small_batch_8_bit_inputs(n, k, r, m, gain, bits):
    err, fmt = _fp8_forward_case(n, k, r, m, seed=23, x_gain=gain, bits=bits)
    assert err <= TOL_Y and fmt == (1 if gain > 1 else 0)


# (no rank of one here: its outputs reach below 2^-14, where rounding to fp16 errs by up to 2^-25 absolute, which the
# element bound, relative to the value, does not cover)
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("n,k,r,m", [(33, 128, 33, 17), (1001, 640, 33, 70), (5000, 1408, 96, 40), (9001, 384, 65, 48),
                                     (20003, 384, 130, 64), (28672, 256, 60, 100)])
def test_small_batch_adapter_term_alone(n, k, r, m, accumulate):
    L, R = wl.make_adapters(n, k, r, 31, 32)
    X = wl.make_activations(m, k, True, 33, 34)
    Lp, Rp = B.slim_pack_adapters(L.to(DEV), R.to(DEV))
    Y0 = Y0h = None
    if accumulate:
        Y0h = (torch.randn(m, n, generator=torch.Generator().manual_seed(9)) * 0.1).to(torch.float16)
        Y0 = Y0h.to(DEV)
    Y = B.slim_lowrank(X.to(DEV), Rp, Lp, n, r, Y=Y0, accumulate=accumulate)
    torch.cuda.synchronize()
    _assert_lowrank_close(Y, X, R, L, Y0=None if Y0h is None else Y0h.numpy())


@pytest.mark.parametrize("bits", [16, 4])
def test_tokens_do_not_leak_into_each_other(bits):
    """Tokens that overflow share tiles, pieces of T and LDS rows with others, which still match the oracle."""
    n, k, r, m = 384, 640, 90, 70
    W, L, R, X = wl.make_layer(_shape(n, k, r), m, seed=24)
    layer = B.compress(W.to(DEV), L.to(DEV), R.to(DEV), adapter_bits=bits)
    if bits == 4:
        L = torch.from_numpy(O.dequantize_adapter(*O.quantize_adapter(L.numpy())))
        R = torch.from_numpy(O.dequantize_adapter(*O.quantize_adapter(R.numpy())))
    bad = [0, 31, 32, 69]
    good = [t for t in range(m) if t not in bad]
    Xg = X.clone()
    Xg[bad] = float("inf")
    Y = B.slim_linear_gemm(layer, Xg.to(DEV))
    torch.cuda.synchronize()
    _assert_layer_close(Y[good], O.compress(W.numpy()), L.numpy(), R.numpy(), X[good], CT_PREFILL + (2 if bits == 4 else 0),
                        "tokens beside infinite ones")


def test_one_workspace_for_every_batch_and_path(decode_override):
    """One workspace, sized for the largest call; batches of all paths in turn (decode, the tile shapes, the large
    tiles), layers of two ranks: no piece of T of an earlier call may pass for this call's."""
    shapes = [_shape(1000, 1152, 70), _shape(5000, 640, 33)]
    data = [wl.make_layer(s, 600, seed=25 + i) for i, s in enumerate(shapes)]
    layers = [_gpu_layer(W, L, R) for W, L, R, _ in data]
    refs = [O.compress(W.numpy()) for W, _, _, _ in data]
    ws = torch.zeros(max(B.slim_workspace_bytes(x, 600) for x in layers), dtype=torch.uint8, device=DEV)
    for i, m in enumerate([64, 600, 64, 17, 300, 40, 600, 33, 512, 64, 64]):
        for (W, L, R, X), layer, ref in zip(data, layers, refs):
            Y = B.slim_linear_gemm(layer, X[:m].to(DEV), workspace=ws)
            torch.cuda.synchronize()
            _assert_layer_close(Y, ref, L.numpy(), R.numpy(), X[:m], CT_PREFILL, f"call {i} m={m}")
    B.slim_workspace_check(ws)


@pytest.mark.parametrize("bits", [16, 4])
def test_a_wait_that_gives_up_is_loud(bits, decode_override):
    """The bounded wait for T, forced from the host to run out (no workgroup makes T, 256 polls; every wavefront
    ends normally): Y is NaN, slim_workspace_check reports it, and the next call on the workspace is correct."""
    shape = _shape(640, 1024, 51)
    W, L, R, X = wl.make_layer(shape, 48, seed=26)
    layer = B.compress(W.to(DEV), L.to(DEV), R.to(DEV), adapter_bits=bits)
    ws = B.alloc_workspace(layer, 48)
    decode_override("wait_test")
    Y = B.slim_linear_gemm(layer, X.to(DEV), workspace=ws)
    torch.cuda.synchronize()
    assert bool(torch.isnan(Y).all())
    with pytest.raises(B.SlimError) as e:
        B.slim_workspace_check(ws)
    assert e.value.status == B.SLIM_ERR_WAIT
    decode_override("auto")
    Y = B.slim_linear_gemm(layer, X.to(DEV), workspace=ws)
    Y2 = B.slim_linear_gemm(layer, X.to(DEV), workspace=B.alloc_workspace(layer, 48))
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2) and bool(torch.isfinite(Y).all())
    B.slim_workspace_check(ws)


@pytest.mark.parametrize("stages", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("fp8", [False, True])
def test_large_tiles_every_stage_count_modulo_six(stages, fp8):
    """Above 512 tokens the main loops are written out for six stages; here on tiles of 128 rows (test_large_tiles has the
    taller ones)."""
    n, k, r, m = 200, 128 * stages, 20, 530
    if fp8:
        err, _ = _fp8_forward_case(n, k, r, m, seed=stages)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=stages)
    assert err <= TOL_Y


# T = X R^T in one launch: as fp16 rows for the 512 x 128 tiles (m > 512) and as pieces (n = 4096: no unit is left for the
# T role), tiles of 16 x 16, 32 x 32, 32 x 64 and 64 x 64 in turn, the last tile of tokens and of ranks partly empty,
# fewer units of inputs than wavefronts and more; the last case is of the tiles of 128 x 128.
T_CASES = [(200, 384, 51, 530), (200, 1792, 200, 530), (200, 256, 510, 545), (200, 128, 992, 577), (200, 1664, 970, 530),
           (4096, 640, 51, 500), (4096, 384, 200, 499), (4096, 256, 530, 481), (4096, 1664, 1100, 500),
           (130, 128, 1024, 2100)]


@pytest.mark.parametrize("kind", ["fp16", "q4", "fp8", "fp8_q4"])
@pytest.mark.parametrize("n,k,r,m", T_CASES)
def test_t_in_one_launch(n, k, r, m, kind):
    bits = 4 if kind.endswith("q4") else 16
    if kind.startswith("fp8"):
        err, _ = _fp8_forward_case(n, k, r, m, seed=27, bits=bits)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=27, bits=bits)
    assert err <= TOL_Y


@pytest.mark.parametrize("n,k,r,m", [(1, 128, 0, 513), (33, 256, 31, 530), (100, 384, 33, 600), (129, 640, 129, 530), (1000, 1152, 300, 540)])
@pytest.mark.parametrize("bits", [16, 4])
def test_large_tiles_with_inputs_divided(n, k, r, m, bits):
    """Tiles of 128 rows with few stages: one stage, odd counts, fewer ranks than a unit, no rows beyond the first."""
    assert _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=28, bits=bits) <= TOL_Y


# one launch for T and Y, with each of the four tile shapes (64 rows x 32 tokens with several tiles of tokens, and more ranks
# than one round of the adapter term)
HELP_CASES = [(512, 512, 51, 17), (33, 128, 33, 31), (700, 4096, 409, 33), (4096, 256, 64, 64), (5000, 1408, 96, 40),
              (2049, 640, 200, 96), (9001, 384, 65, 48), (20003, 384, 130, 64)]


@pytest.mark.parametrize("kind", ["fp16", "q4", "fp8", "fp8_q4"])
@pytest.mark.parametrize("n,k,r,m", HELP_CASES)
def test_a_workgroup_whose_wait_runs_out_makes_t_itself(n, k, r, m, kind, decode_override):
    """The T role makes nothing (forced from the host), as if other work on the chip kept it from being dispatched: the waits run out
    after 256 polls, and every workgroup makes T of its tokens and starts again.  The bounds are the usual ones."""
    decode_override("wait_test", 16)
    bits = 4 if kind.endswith("q4") else 16
    if kind.startswith("fp8"):
        err, _ = _fp8_forward_case(n, k, r, m, seed=29, bits=bits)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=29, bits=bits)
    assert err <= TOL_Y


def test_a_forced_wait_leaves_the_same_bits_and_no_error(decode_override):
    shape = _shape(5000, 1408, 96)
    W, L, R, X = wl.make_layer(shape, 40, seed=30)
    layer = _gpu_layer(W, L, R)
    ws = B.alloc_workspace(layer, 40)
    Y = B.slim_linear_gemm(layer, X.to(DEV), workspace=ws)
    decode_override("wait_test", 16)
    Y2 = B.slim_linear_gemm(layer, X.to(DEV), workspace=ws)
    Z2 = B.slim_lowrank(X.to(DEV), layer.R, layer.L, 5000, 96, workspace=ws)
    decode_override("auto")
    Z = B.slim_lowrank(X.to(DEV), layer.R, layer.L, 5000, 96, workspace=ws)
    torch.cuda.synchronize()
    B.slim_workspace_check(ws)
    assert torch.equal(Y, Y2) and torch.equal(Z, Z2)


def test_overlapping_small_batch_calls():
    """Small-batch calls on four streams at a time, each taking whole compute units and waiting for its own T, in a new
    order each time: every result is the one of the call alone, and no wait was lost."""
    m = 40
    shapes = [(5000, 1408, 96), (9001, 384, 65), (4096, 1024, 102), (5000, 1408, 200)]
    streams = [torch.cuda.Stream(device=DEV) for _ in shapes]
    jobs = []
    for i, (n, k, r) in enumerate(shapes):
        W, L, R, X = wl.make_layer(_shape(n, k, r), m, seed=40 + i)
        layer, Xd = _gpu_layer(W, L, R), X.to(DEV)
        alone = B.slim_linear_gemm(layer, Xd)
        jobs.append((layer, Xd, alone, B.alloc_workspace(layer, m), [torch.empty_like(alone) for _ in range(12)]))
    torch.cuda.synchronize()
    for call in range(12):
        for i in range(len(jobs)):
            j = (i + call) % len(jobs)
            layer, Xd, _, ws, outs = jobs[j]
            with torch.cuda.stream(streams[j]):
                B.slim_linear_gemm(layer, Xd, Y=outs[call], workspace=ws)
    torch.cuda.synchronize()
    for layer, Xd, alone, ws, outs in jobs:
        B.slim_workspace_check(ws)
        assert all(torch.equal(alone, y) for y in outs)


@pytest.mark.parametrize("kind", ["fp16", "q4", "fp8", "fp8_q4"])
@pytest.mark.parametrize("n,k,r,m,t_kind", [
    (28672, 1024, 60, 200, (3, 3)), (200, 512, 51, 530, (0, 0)), (200, 1024, 200, 1100, (1, 1)), (200, 1152, 130, 2600, (1, 1)),
    (200, 2048, 200, 4000, (2, 2)), (100, 128, 1024, 3000, (4, 4)), (60, 8192, 800, 1500, (4, 4))])
def test_every_kind_of_t_product(n, k, r, m, t_kind, kind):
    """T as rows for the large tiles by each of its kernels (the rule's choice is checked, so that a later rule does not
    take the coverage away): token tiles that the dies do not divide evenly, the last tiles partly empty."""
    from test_dispatch_rules import _t_kind
    bits = 4 if kind.endswith("q4") else 16
    assert _t_kind(B.slim_rank_pad(r), m, k, bits == 4, True) == t_kind[bits == 4]
    if kind.startswith("fp8"):
        err, _ = _fp8_forward_case(n, k, r, m, seed=31, bits=bits)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=31, bits=bits)
    assert err <= TOL_Y


@pytest.mark.parametrize("bits,xf", [(16, 0), (16, 1), (16, 2), (4, 0), (4, 1), (4, 2)])
@pytest.mark.parametrize("m,r,k,splits", [
    (1, 1, 128, 1), (127, 32, 256, 2), (128, 128, 384, 4), (129, 129, 640, 8), (260, 150, 1152, 2), (1100, 300, 512, 1), (1025, 33, 2048, 8),
    (130, 40, 33024, 1)])
def test_t_in_tiles_of_128(m, r, k, splits, bits, xf):
    """The tiles of 128 ranks x 128 tokens alone: one and several tiles, their remainders on both sides, ranges of the inputs that are uneven
    (five groups of 128 on two and eight) or empty, and more inputs than the 4-bit scales in LDS hold.  T is a sum in fp32, rounded to fp16 once."""
    g = torch.Generator().manual_seed(k + m)
    Rw = torch.randn(r, k, generator=g).half() * 0.05
    L = torch.zeros(8, r, dtype=torch.half)
    rp = B.slim_rank_pad(r)
    if bits == 4:
        q = B.slim_pack_adapters_q4(L.to(DEV), Rw.to(DEV))
        Rq, Rs, R = q[2], q[3], None
        codes, scales = B.slim_unpack_adapters_q4(Rq, Rs, r, k)
        R64 = (codes.half().cpu() * scales.half().cpu().repeat_interleave(128, 1)[:, :k]).double()
    else:
        R, Rq, Rs, R64 = B.slim_pack_adapters(L.to(DEV), Rw.to(DEV))[1], None, None, Rw.double()
    if xf:
        f8 = torch.float8_e4m3fn if xf == 1 else torch.float8_e5m2
        Xc = torch.randn(m, k, generator=g).to(f8)
        X64, X, scale = Xc.double(), Xc.view(torch.uint8).to(DEV), torch.tensor([0.625], device=DEV)
    else:
        Xh = torch.randn(m, k, generator=g).half()
        X64, X, scale = Xh.double(), Xh.to(DEV), torch.tensor([1.0], device=DEV)
    T = torch.full((m, rp), float("nan"), dtype=torch.half, device=DEV)
    P = torch.full((splits * m * rp,), float("nan"), device=DEV)
    vp, i32 = ctypes.c_void_p, ctypes.c_int
    f = B.lib()._ZN4slim14launch_t_splitEPKDF16_iPKfiiS1_PKhS1_iiPDF16_PfiP12ihipStream_t
    f.argtypes = [vp, i32, vp, i32, i32, vp, vp, vp, i32, i32, vp, vp, i32, vp]
    ptr = lambda t: None if t is None else t.data_ptr()
    assert f(ptr(X), xf, ptr(scale), m, k, ptr(R), ptr(Rq), ptr(Rs), r, rp, ptr(T), ptr(P), splits, torch.cuda.current_stream().cuda_stream) == 0
    s = float(scale)
    ref, size = s * (X64 @ R64.T), s * (X64.abs() @ R64.abs().T)
    # fp32: a rounding for each of at most k / 16 + 16 partial sums, of at most `size`; fp16: half a unit of the result
    bound = (k / 16 + 16) * 2.0 ** -24 * size
    bound = bound + 2.0 ** -11 * (ref.abs() + bound) + 2.0 ** -25
    got = T.double().cpu()
    assert bool(((got[:, :r] - ref).abs() <= bound).all())
    assert bool((got[:, r:] == 0).all())


def _tile_height(n, m):
    """Rows of a tile / 128 of slim_linear_gemm's large tiles, where one launch has them all."""
    tiles, whole, _ = B.slim_gemm_tile_order(n, m)
    assert whole in (0, tiles)
    return 4 if whole else 2 if 4 * tiles > 256 else 1


@pytest.mark.parametrize("kind", ["fp16", "q4", "fp8", "fp8_q4"])
@pytest.mark.parametrize("groups,stages", [(1, s) for s in (1, 2, 3, 4, 5, 6, 7)] + [(2, s) for s in (18, 19, 21, 22, 23, 25, 27)])
@pytest.mark.parametrize("height,n,m", [(4, 5120, 1663), (2, 5120, 870), (1, 200, 530)])
def test_large_tiles(height, n, m, groups, stages, kind):
    """The main loops of the tiles of 512, 256 and 128 rows, written out for six stages of 128 inputs, on stage counts of every
    remainder, below and above one pass; on the lower two by one group of wavefronts and by two (with odd counts, where the second
    group's last stage does not exist), whose share of the stages has every remainder modulo six too.  What
    tile and how many groups a size gets is checked, so that a later rule does not take the coverage away."""
    from test_dispatch_rules import _two_groups
    k, r = 128 * stages, 20
    assert _tile_height(n, m) == height
    assert _two_groups(k, B.slim_rank_pad(r), False) == (groups == 2)
    if kind.startswith("fp8") and groups == 2:
        k -= 128 * 6                    # 8-bit inputs: two groups from ten stages on
        assert _two_groups(k, B.slim_rank_pad(r), True)
    rows = np.unique(np.r_[0, n - 1, np.random.default_rng(stages).integers(0, n, 40)])
    bits = 4 if kind.endswith("q4") else 16
    if kind.startswith("fp8"):
        err, _ = _fp8_forward_case(n, k, r, m, seed=stages, bits=bits, rows=rows)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=stages, bits=bits, rows=rows)
    assert err <= TOL_Y


@pytest.mark.parametrize("n,k,r,m", [(700, 1152, 70, 40), (4096, 640, 51, 500), (4096, 640, 200, 600)])
def test_captured_calls_replay_correctly(n, k, r, m):
    """slim_linear_gemm on fp16 and 4-bit adapters, slim_linear_gemm_fp8 and slim_lowrank captured into one graph, on
    one workspace: T in the same launch, in one of its own (no unit left for the T role), and as rows.  Every replay gets
    new inputs, with eager calls on the same workspace and a synchronization in between, and equals the eager results."""
    W, L, R, X = wl.make_layer(_shape(n, k, r), m, seed=60)
    layers = [B.compress(W.to(DEV), L.to(DEV), R.to(DEV), adapter_bits=bits) for bits in (16, 4)]
    ws = torch.zeros(max(B.slim_workspace_bytes(x, m) for x in layers), dtype=torch.uint8, device=DEV)
    Xd = X.to(DEV)
    codes, info = torch.empty(m, k, dtype=torch.uint8, device=DEV), torch.empty(2, device=DEV)
    qws = torch.empty(1024, dtype=torch.uint8, device=DEV)
    out = [torch.empty(m, n, dtype=torch.float16, device=DEV) for _ in range(4)]

    def calls(out, ws):
        for i in (0, 1):
            B.slim_linear_gemm(layers[i], Xd, Y=out[i], workspace=ws)
        B.slim_input_quant_fp8(Xd, Xq=False, info=info, workspace=qws, codes=codes)
        B.slim_linear_gemm_fp8(layers[1], codes, info, 0, Y=out[2], workspace=ws)
        B.slim_lowrank(Xd, layers[0].R, layers[0].L, n, r, Y=out[3], workspace=ws)

    calls(out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls(out, ws)
    own = torch.zeros_like(ws)
    for replay in range(4):
        Xd.copy_(X.to(DEV).roll(replay, 0) * (1 + replay / 4))
        graph.replay()
        torch.cuda.synchronize()
        got = [y.clone() for y in out]
        want = [torch.empty_like(y) for y in out]
        calls(want, own if replay % 2 else ws)
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert torch.equal(g, w)
    B.slim_workspace_check(ws)


# T in tiles of 32 tokens beside each of the four tile shapes, one per workgroup and two, token counts that end in either half of a tile
T32_CASES = [(7452, 256, 243, 31), (1604, 1024, 102, 109), (1485, 1536, 148, 189), (3127, 384, 230, 150), (2244, 384, 224, 343)]


@pytest.mark.parametrize("help_t", [False, True])
@pytest.mark.parametrize("kind", ["fp16", "q4", "fp8", "fp8_q4"])
@pytest.mark.parametrize("n,k,r,m", T32_CASES)
def test_t_in_tiles_of_32_tokens(n, k, r, m, kind, help_t, decode_override):
    """By the T role, and by workgroups whose wait runs out.  The bounds are the usual ones."""
    from test_dispatch_rules import _mid_plan
    assert _mid_plan(n, k, B.slim_rank_pad(r), m, True, kind.endswith("q4"), kind.startswith("fp8"))[1] == 32
    if help_t:
        decode_override("wait_test", 16)
    bits = 4 if kind.endswith("q4") else 16
    if kind.startswith("fp8"):
        err, _ = _fp8_forward_case(n, k, r, m, seed=33, bits=bits)
    else:
        err = _forward_case(_shape(n, k, r), m, B.slim_linear_gemm, seed=33, bits=bits)
    assert err <= TOL_Y
