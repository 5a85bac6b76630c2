"""How many products of the adapter computation follow on one another before a block is orthonormalised: the library's own rule
(host code), by itself and in a replay of the iteration in binary32 (products of two fp16 parts each, Cholesky QR, columns that
are only scaled in between) against binary64 with every block orthonormal."""
import ctypes

import numpy as np
import pytest

from paper_2410_09615_amd import binding as B


def _run(done, h, pmax, pmin):
    f = B.lib()._ZN4slim8orth_runEiiff
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_float], ctypes.c_int
    return f(done, h, pmax, pmin)


def _due(h, run, last):
    f = B.lib()._ZN4slim8orth_dueEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    return f(h, run, last)


@pytest.mark.parametrize("spread", [0.0, 1.0, 9.0, 29.0, 31.0, 99.0, 101.0, 255.0, 999.0, 1001.0, 9999.0, 1.1e4, 1e9, float("inf"), float("nan")])
def test_a_run_is_no_longer_than_its_span_allows(spread):
    """Rounding of 2e-7 of a column grows by the ratio of the singular values, the root of the span, with each product: below 0.2
    at the end of a run; one product is always allowed."""
    for h in (0, 1, 3, 6, 7, 8, 100):
        seen, todo = set(), [0]
        while todo:
            done = todo.pop()
            run = _run(done, h, spread, 1.0)
            assert 1 <= run <= (8 if h >= 7 else 2) and run <= max(1, 2 * done)
            assert run == 1 or (spread <= 1e4 and 2e-7 * np.sqrt(spread) ** run <= 0.2)
            if run not in seen:
                seen.add(run)
                todo.append(run)
    # no block with a pivot above the floor (a matrix of zeros)
    assert _run(0, 0, 0.0, float("inf")) == 1 and 1 <= _run(8, 31, 0.0, float("inf")) <= 8


@pytest.mark.parametrize("last", [2, 4, 6, 8, 10, 12, 14, 16, 32, 34, 2000])
@pytest.mark.parametrize("run", [1, 2, 4, 8])
def test_the_last_run_is_short(run, last):
    for first in (1, run):
        h, steps = 0, []
        while h < last:
            due = _due(h, first if h == 0 else run, last)
            assert h < due <= last and due - h <= 8
            assert due < last or due - h <= 4
            h, steps = due, steps + [due - h]
        assert sum(steps) == last and steps[0] == min(first, last - 4 if last > 4 else last)


@pytest.mark.parametrize("l", [32, 64, 96, 256, 416, 640, 832, 992, 1024])
@pytest.mark.parametrize("rows", [1, 31, 64, 65, 1000, 4096, 4097, 28672, 28673, 100000, (1 << 22) - 32, 1 << 22, (1 << 22) + 1, (1 << 24) - 4096])
def test_ranges_of_rows_of_a_gram_matrix(rows, l):
    """They are the rows, fit the workspace's partial tiles, and a wavefront's quarter of one, with the rows it reads ahead, has 32-bit
    offsets in bytes; none is much longer than 4096 rows while there is room for more."""
    f, each = B.lib()._ZN4slim11gram_rangesEiiPi, ctypes.c_int()
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    n, nb = f(rows, l, ctypes.byref(each)), -(-l // 64)
    tiles = nb * (nb + 1) // 2
    assert (n - 1) * each.value < rows <= n * each.value and each.value % 32 == 0
    assert 1 <= n and n * tiles <= 640
    assert (each.value // 4 + 64) * l * 4 < 1 << 32
    most = 640 // tiles if 640 // tiles <= 8 else 640 // tiles // 8 * 8
    assert each.value <= 4096 * 9 // 8 + 32 or n == most          # (more than eight ranges are a multiple of eight)


@pytest.mark.parametrize("nb", range(1, 17))
@pytest.mark.parametrize("room", [1, 2, 57])
def test_a_factorisation_ends_with_room_for_few_workgroups(nb, room):
    """A workgroup per strip, started in the order of their index as those before them end, beside the one of the diagonal tiles: with room
    for a single strip all of them end.  What waits for what is replayed from the order in which the library has the strips."""
    f, out = B.lib()._ZN4slim8strip_atEiiPiS0_S0_, [ctypes.c_int() for _ in range(3)]
    f.argtypes, f.restype = [ctypes.c_int] * 2 + [ctypes.c_void_p] * 3, None
    strips = []
    for i in range(4 * (nb * (nb + 1) // 2 - 1)):
        f(i, nb, *[ctypes.byref(v) for v in out])
        strips.append(tuple(v.value for v in out))
    assert sorted(strips) == sorted((I, j, q) for I in range(nb) for j in range(I + 1) for q in range(4) if I > 0)
    handed, factor, diagonal = set(), set(), 0        # strips handed to the chain, strips of the factor, diagonal tiles that are done

    def ends(I, j, q):
        columns = range(j - 1 if I == j else j)
        if not all((I, K, q) in factor and all((j, K, w) in factor for w in range(4)) for K in columns):
            return False
        if I <= j + 1:
            handed.add((I, j, q))
        if I > j and diagonal > j:
            factor.add((I, j, q))
        return I == j or diagonal > j

    waiting, running = list(strips), []
    while waiting or running or diagonal < nb:
        before = len(handed), len(factor), diagonal, len(waiting)
        while diagonal < nb and all(diagonal == 0 or ((diagonal, diagonal, q) in handed and (diagonal, diagonal - 1, q) in handed) for q in range(4)):
            diagonal += 1
        running += [waiting.pop(0) for _ in range(min(room - len(running), len(waiting)))]
        running = [s for s in running if not ends(*s)]
        assert (len(handed), len(factor), diagonal, len(waiting)) != before, "nothing that runs can go on"


def _orth(Y):
    """Cholesky QR in binary32, columns in order: (block, largest pivot, smallest pivot)."""
    A = (Y.T @ Y).astype(np.float32)
    M = np.eye(len(A), dtype=np.float32)
    d = np.ones(len(A), np.float32)
    for c in range(len(A)):
        d[c] = A[c, c]
        M[c + 1:, c] = A[c + 1:, c] / d[c]
        A[c + 1:, c + 1:] -= np.outer(M[c + 1:, c], A[c + 1:, c])
    out = np.array(Y.T)
    for c in range(len(A)):
        out[c + 1:] -= np.outer(M[c + 1:, c], out[c])
    return (out / np.sqrt(d)[:, None]).T.astype(np.float32), float(d.max()), float(d.min())


def _ruled(done, h, pmax, pmin, last):
    run = _run(done, h, pmax, pmin)
    return run, _due(h, run, last)


def _pairs(done, h, pmax, pmin, last):
    """Two products in a row at most, while the pivots span no more than 1e4."""
    run = 2 if h % 2 and pmax <= 1e4 * pmin else 1
    return run, h + run


def _replay(S, Z, iters, rule):
    S, last = S.astype(np.float32), 2 * iters
    Y, due, run, blocks = S @ Z.astype(np.float32), 0, 0, 0
    for h in range(last):
        if h >= due:
            b, pmax, pmin = _orth(Y)
            run, due = rule(run, h, pmax, pmin, last)
            blocks += 1
        else:
            b = np.ldexp(Y, -np.frexp(np.abs(Y).max(0))[1])
        v = b * np.float32(64)
        hi = v.astype(np.float16).astype(np.float32)
        b = (hi + (v - hi).astype(np.float16).astype(np.float32)) / np.float32(64)
        Y = S.T @ b if h % 2 == 0 else S @ b
    Q, _, _ = _orth(Y)
    return _orth(Q)[0].astype(np.float64), blocks


def _spectrum(kind, n, k, r, rng):
    if kind.startswith("channels"):                              # r channels that span a factor above the others
        x = np.ones(k)
        x[rng.permutation(k)[:r]] = float(kind[8:]) ** (1 - np.arange(r) / r)
        return rng.standard_normal((n, k)) * 0.02 * x
    U, _ = np.linalg.qr(rng.standard_normal((n, n)))
    V, _ = np.linalg.qr(rng.standard_normal((k, n)))
    s = np.ones(n)
    if kind.startswith("one above"):
        s[0], s[r:] = float(kind[9:]), 0.9
    elif kind == "geometric":
        s[:r], s[r:] = 6.0 ** (np.arange(r)[::-1] / r), 0.3
    else:
        s = np.arange(1.0, n + 1) ** -0.5
    return U * s @ V.T


@pytest.mark.parametrize("kind", ["channels1", "channels8", "one above 3", "one above 6", "one above 10", "geometric", "power"])
@pytest.mark.parametrize("iters", [2, 4, 6, 8, 16])
def test_l_spans_what_it_does_with_two_products_in_a_row(kind, iters):
    """Distance of L, before it is rounded to fp16, from the span of the exact iterate: some units of binary32 rounding (2e-6 to 1e-5)
    with two products in a row, and in replays of 16 kinds of spectra, 1 to 24 rounds, up to 1.5 times that with the rule; asked
    is twice.  (Runs of four from the third product on: up to 110 times; a last run of eight: 41 times.)"""
    n, k, r = 192, 256, 26
    rng = np.random.default_rng(iters)
    S, Z = _spectrum(kind, n, k, r, rng), rng.uniform(-1, 1, (k, r))
    Q, _ = np.linalg.qr(S @ Z)
    for _ in range(iters):
        Q, _ = np.linalg.qr(S @ np.linalg.qr(S.T @ Q)[0])

    def off(P):
        return np.linalg.norm(P - Q @ (Q.T @ P))

    pairs, most = _replay(S, Z, iters, _pairs)
    ruled, blocks = _replay(S, Z, iters, _ruled)
    assert off(ruled) <= 2 * off(pairs)
    assert blocks <= most
    assert np.max(np.abs(ruled.T @ ruled - np.eye(r))) <= 1e-5
