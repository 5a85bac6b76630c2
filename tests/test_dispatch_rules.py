"""Host logic: which kernel a call is sent to.  The times are measured ones (us, MI355X, products alone in a
row), those of the sizes where one rule or another once chose badly; asked is that the kind chosen takes at most a tenth longer than
the best of them (a fifth where said so), which is what the estimates behind the rule are good for.  (The rules ask the device for its
compute units; without one they plan for 256.)"""
import ctypes

import pytest

from paper_2410_09615_amd import binding as B


def _t_kind(rank_pad, m, k, q4, split):
    f = B.lib()._ZN4slim6t_kindEiiibb
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool] * 2
    return f(rank_pad, m, k, q4, split)


NO = float("inf")


@pytest.mark.parametrize("q4,k,rank_pad,m,us", [
    (False, 512, 64, 128, [4.4, 4.4, 5.5, 3.9, 7.9]),
    (False, 2048, 32, 2048, [5.1, 6.5, 8.4, 16.2, 10.1]),
    (False, 4096, 128, 1500, [8.0, 9.5, 12.9, 21.1, 13.9]),
    (False, 8192, 64, 800, [10.6, 14.8, 20.5, 20.3, 12.8]),
    (False, 8192, 416, 1000, [26.0, 20.2, 25.0, NO, 19.6]),
    (False, 8192, 512, 800, [26.5, 20.4, 26.2, NO, 19.2]),
    (False, 8192, 832, 512, [27.4, 21.8, 27.6, NO, 18.6]),
    (False, 11008, 1120, 64, [35.7, 49.6, 33.5, 17.6, 14.7]),
    (False, 11008, 416, 2048, [64.7, 49.9, 33.3, NO, 30.1]),
    (False, 13824, 128, 3000, [42.0, 31.5, 39.9, NO, 23.1]),
    (False, 13824, 608, 600, [40.8, 59.1, 41.4, NO, 21.2]),
    (False, 28672, 224, 2048, [78.3, 62.2, 74.6, NO, 35.7]),
    (False, 28672, 832, 200, [54.9, 65.7, 80.2, 62.8, 26.4]),
    (False, 28672, 832, 128, [53.9, 62.2, 76.9, 42.9, 27.0]),
    (False, 28672, 832, 256, [55.4, 64.8, 79.8, NO, 28.1]),
    (False, 28672, 1408, 48, [85.4, 107.4, 75.9, 41.1, 24.0]),
    (True, 4096, 512, 2048, [28.6, 21.8, 17.9, NO, 25.7]),
    (True, 8192, 832, 1000, [47.8, 37.8, 29.7, NO, 31.9]),
    (True, 11008, 128, 2048, [18.4, 26.9, 39.5, NO, 23.2]),
    (False, 2048, 1120, 2048, [NO, NO, 26.4, NO, 16.7]),
    (False, 8192, 832, 4096, [NO, NO, 97.8, NO, 60.5]),
    (False, 18560, 480, 596, [NO, 40.8, NO, NO, 22.8]),
    (False, 27264, 64, 2105, [37.7, NO, NO, NO, 28.2]),
    (False, 28672, 832, 4096, [NO, NO, 337.4, NO, 220.4]),
    (True, 11008, 1024, 4096, [NO, NO, 152.4, NO, 113.2]),
    (True, 28672, 832, 500, [NO, 64.5, NO, NO, 43.8]),
])
def test_the_kind_of_t_product(q4, k, rank_pad, m, us):
    """us: kinds 0 to 4, the last (tiles of 128 x 128) at the number of ranges that t_splits() takes.  Its estimate is a tenth above what it takes, so that of
    two about as fast the one launch is taken: it may be a fifth slower than kind 4, a tenth than another of one launch.  Up to 128 tokens kind 4
    is not taken."""
    kind = _t_kind(rank_pad, m, k, q4, True)
    assert us[kind] <= 1.1 * min(us[:4]) and (m <= 128 or us[kind] <= 1.2 * us[4])
    assert kind != 4 or m > 128
    assert us[_t_kind(rank_pad, m, k, q4, False)] <= 1.2 * min(us[:4])


@pytest.mark.parametrize("q4,k,rank_pad,m,us", [
    (False, 2048, 1120, 2048, {1: 16.7, 2: 28.0, 4: 33.6}),
    (False, 4096, 416, 4096, {1: 24.9, 2: 24.8, 4: 32.9}),
    (False, 5120, 512, 1000, {1: 32.3, 2: 22.1, 4: 18.8, 8: 20.1}),
    (False, 8192, 416, 1000, {1: 42.4, 2: 27.4, 4: 20.3, 8: 19.6}),
    (False, 8192, 832, 2048, {1: 43.6, 2: 37.1, 4: 42.8}),
    (False, 8192, 832, 4096, {1: 60.5, 2: 70.4}),
    (False, 11008, 416, 1000, {1: 59.0, 2: 35.1, 4: 23.6, 8: 20.8}),
    (False, 11008, 416, 2048, {1: 58.6, 2: 36.6, 4: 30.1, 8: 36.6}),
    (False, 13824, 128, 3000, {1: 72.2, 2: 42.7, 4: 27.7, 8: 23.1}),
    (False, 28672, 224, 2048, {1: 137.2, 2: 74.4, 4: 44.9, 8: 35.7}),
    (False, 28672, 832, 1000, {1: 147.2, 2: 81.3, 4: 55.9, 8: 63.0}),
    (False, 28672, 832, 4096, {1: 220.4, 2: 239.6}),
    (True, 4096, 512, 2048, {1: 40.7, 2: 29.9, 4: 25.7, 8: 32.0}),
    (True, 8192, 832, 1000, {1: 74.7, 2: 44.6, 4: 31.9, 8: 36.7}),
    (True, 11008, 1024, 4096, {1: 113.2, 2: 124.8}),
    (True, 28672, 832, 500, {1: 247.8, 2: 130.2, 4: 70.7, 8: 43.8}),
])
def test_the_ranges_of_t_in_tiles_of_128(q4, k, rank_pad, m, us):
    """us: by the number of ranges, as many as the workspace has room for."""
    f, room = B.lib()._ZN4slim8t_splitsEiiib, B.lib()._ZN4slim13gemm_t_splitsEiii
    f.argtypes, room.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool], [ctypes.c_int] * 3
    assert max(us) == room(m, rank_pad, k)
    assert us[f(rank_pad, m, k, q4)] <= 1.1 * min(us.values())


def test_the_kind_of_t_product_is_always_one():
    for k in (128, 4096, 28672):
        for rank_pad in (32, 1024, 4096):
            for m in (17, 1000, 100000):
                for q4 in (False, True):
                    assert 0 <= _t_kind(rank_pad, m, k, q4, True) <= 4
                    assert 0 <= _t_kind(rank_pad, m, k, q4, False) <= 3


def _two_groups(k, rank_pad, fp8):
    f = B.lib()._ZN4slim10two_groupsEiib
    f.argtypes = [ctypes.c_int] * 2 + [ctypes.c_bool]
    f.restype = ctypes.c_bool
    return f(k, rank_pad, fp8)


@pytest.mark.parametrize("fp8,k,rank_pad,ratio", [
    (False, 128, 0, 1.12), (False, 512, 0, 1.09), (False, 1024, 0, 1.05), (False, 1024, 128, 1.05), (False, 2048, 64, 1.02),
    (False, 4096, 0, 0.95), (False, 4096, 416, 0.94), (False, 8192, 832, 0.94), (False, 11008, 0, 0.94),
    (True, 128, 0, 1.10), (True, 512, 64, 1.05), (True, 1536, 0, 0.96), (True, 2048, 64, 0.95), (True, 4096, 416, 0.88)])
def test_two_groups_of_wavefronts_where_they_pay(fp8, k, rank_pad, ratio):
    """ratio: time of a call with two groups over that with one, measured (mean of calls on 512 to 28672 rows)."""
    assert _two_groups(k, rank_pad, fp8) == (ratio < 1.0)


def _mid_plan(n, k, rank_pad, m, weight_term, q4=False, fp8=False):
    f = B.lib()._ZN4slim8mid_planEiiiiibbb
    f.argtypes, f.restype = [ctypes.c_int] * 5 + [ctypes.c_bool] * 3, ctypes.c_uint64
    v = f(n, k, rank_pad, m, 256, weight_term, q4, fp8)
    return ctypes.c_int32(v & 0xFFFFFFFF).value, v >> 32


@pytest.mark.parametrize("n,k,r,m,us", [
    (2244, 3968, 224, 343, {(-1, 0): 32.0, (3, 0): 25.8, (3, 32): 17.6}),
    (7452, 2432, 243, 31, {(0, 0): 12.0, (0, 16): 10.1, (0, 32): 8.6, (1, 0): 11.8, (1, 16): 8.2, (1, 32): 8.8, (2, 16): 10.0, (2, 32): 10.0}),
    (1375, 3584, 137, 126, {(0, 0): 13.2, (0, 16): 11.4, (0, 32): 9.8, (1, 16): 9.3, (1, 32): 10.2, (2, 16): 12.4, (2, 32): 12.5}),
    (1540, 4096, 154, 98, {(0, 0): 13.1, (0, 32): 13.9, (1, 16): 9.3, (1, 32): 10.1, (2, 16): 12.3}),
    (3127, 2304, 230, 156, {(1, 0): 19.4, (2, 0): 15.2, (2, 16): 12.3, (2, 32): 11.2, (3, 16): 15.0}),
    (12523, 7040, 704, 36, {(1, 0): 41.0, (2, 0): 33.0, (2, 16): 29.8, (2, 32): 27.7, (3, 16): 36.8}),
    (11008, 8192, 819, 48, {(1, 0): 41.2, (2, 0): 32.9, (2, 16): 25.2, (2, 32): 26.0, (3, 16): 35.4}),
    (5120, 5120, 512, 48, {(0, 0): 23.0, (1, 0): 17.2, (1, 16): 11.7, (1, 32): 13.2, (2, 16): 15.7}),
    (13056, 3200, 320, 148, {(-1, 0): 29.9, (3, 0): 39.7}),
    (12572, 3072, 499, 20, {(1, 16): 10.6, (1, 32): 11.8}),
    (12572, 8192, 819, 20, {(1, 16): 25.0, (1, 32): 21.8})])
def test_the_plan_of_small_batches(n, k, r, m, us):
    """Tile and T of whole layers: the plan taken is within a tenth of the best one measured."""
    assert us[_mid_plan(n, k, B.slim_rank_pad(r), m, True)] <= 1.1 * min(us.values())


@pytest.mark.parametrize("kind,n,k,r,m,us", [
    # few workgroups with a second tile of 16 tokens, and more
    ("gemm", 2610, 3200, 261, 74, {(1, 16): 10.2, (1, 32): 11.2}),
    ("gemm q4", 2688, 4736, 268, 79, {(1, 16): 12.2, (1, 32): 12.1}),
    ("gemm", 4399, 4352, 435, 56, {(1, 16): 11.7, (1, 32): 12.5}),
    ("gemm", 5888, 2816, 281, 38, {(1, 16): 9.1, (1, 32): 10.2}),
    ("gemm", 2560, 2432, 243, 106, {(1, 16): 9.6, (1, 32): 8.6}),
    ("gemm q4", 2304, 8064, 230, 100, {(1, 16): 16.9, (1, 32): 14.9}),
    ("gemm", 3031, 6656, 303, 96, {(1, 16): 15.4, (1, 32): 13.9}),
    ("lowrank", 9600, 9728, 960, 27, {(1, 16): 19.5, (1, 32): 21.4}),
    ("lowrank", 12288, 5888, 588, 22, {(1, 16): 14.4, (1, 32): 15.2}),
    ("lowrank", 4992, 9984, 499, 55, {(1, 16): 19.5, (1, 32): 17.1}),
    # two tiles of 32 tokens, or the next tile of Y
    ("gemm", 4096, 7168, 409, 86, {(2, 16): 18.8, (1, 32): 20.5}),
    ("gemm", 2304, 3328, 230, 153, {(2, 32): 11.4, (2, 16): 11.4, (1, 32): 13.0}),
    ("fp8 q4", 4864, 1024, 102, 83, {(2, 16): 8.2, (1, 32): 10.1}),
    ("fp8", 3840, 5120, 384, 86, {(2, 16): 15.1, (1, 32): 11.6}),
    ("gemm q4", 3744, 9344, 374, 69, {(2, 16): 26.4, (1, 16): 19.1}),
    ("gemm", 9600, 896, 89, 69, {(3, 16): 8.3, (2, 32): 9.5}),
    ("fp8 q4", 3456, 1024, 102, 210, {(3, 16): 9.6, (2, 32): 10.8}),
    ("fp8", 13184, 6400, 640, 33, {(3, 16): 27.9, (2, 32): 19.6}),
    ("gemm", 7101, 6016, 601, 86, {(3, 16): 29.0, (2, 32): 22.5}),
    # 4-bit adapters on long sums
    ("fp8 q4", 2048, 9856, 204, 205, {(2, 16): 22.6, (2, 32): 25.6}),
    ("fp8 q4", 4951, 7296, 495, 90, {(2, 16): 22.3, (2, 32): 24.8}),
    ("fp8 q4", 640, 1152, 64, 432, {(2, 16): 9.9, (2, 32): 8.9})])
def test_the_plan_by_ranks_inputs_and_types(kind, n, k, r, m, us):
    """The two or three plans that a rule decides between: the faster one, or one within 6 %."""
    plan = _mid_plan(n, k, B.slim_rank_pad(r), m, kind != "lowrank", "q4" in kind, "fp8" in kind)
    assert us[plan] <= 1.06 * min(us.values())


def test_the_plan_of_the_adapter_term_alone():
    assert _mid_plan(4096, 4096, 416, 128, False) == (1, 0)        # 12.1 us; in one launch 12.7
    assert _mid_plan(2679, 896, 96, 203, False) == (2, 32)        # 8.9 us; two tiles of 16 tokens 10.2
    assert _mid_plan(2016, 2176, 224, 96, False) == (1, 16)        # 8.2; on the smallest tile 10.4
    assert _mid_plan(18662, 2560, 256, 64, False) == (3, 16) and _mid_plan(28672, 8192, 832, 400, False)[0] == -1
