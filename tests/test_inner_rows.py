"""Matrices whose large rows cancel in some columns and add up in others.

The walks over pairs of columns form products from differences between the signs
of a few inner rows.  Where inner rows dominate a pair's columns and cancel there,
a difference loses the digits of a small product that other columns make count,
so such a matrix has its products formed from the column sums.  Two rows S times
the others cancel in columns 0 and 1 and add up in 2 and 3, as the last rows of a
matrix (inner rows), as one inner row and another one, and as two others; two
more rows do so in columns of their own.

A column sum holding entries of size S is rounded at 2^-53 S, beside sums of order
one: four such columns, each a few roundings, make the bound 16 * 2^-53 S on top
of the reported estimate, with the oracle in double-double as the reference.  In
the leave-one-column-out walk an inner row is added to a sum and taken off it
twice, so its sums hold 2 S and its bound is twice as wide."""
import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I
from tests import test_minor_pairs
from tests.test_minor_pairs import exe as minors_exe  # noqa: F401  (a fixture)
from tests.test_pair_walk import emulate, exe, rel  # noqa: F401  (exe is a fixture)

U = 2.0 ** -53
KINDS = ["both", "one", "none", "crossed"]


def matrix(n, S, kind, seed=0, rows=None):
    """n columns, `rows` (n) rows; the scaled ones are the last two, the last and
    the third, or the second and third."""
    rows = rows or n
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((rows, n)) + 1j * rng.standard_normal((rows, n))
    last = rows - 1
    if kind == "crossed":  # columns 0 and 2 by the last rows, 1 and 3 by two others
        A[last - 1, [0, 2]] *= S
        A[last, 0], A[last, 2] = -A[last - 1, 0], A[last - 1, 2]
        A[1, [1, 3]] *= S
        A[2, 1], A[2, 3] = -A[1, 1], A[1, 3]
        return A
    a, b = {"both": (last - 1, last), "one": (2, last), "none": (1, 2)}[kind]
    A[a, :4] *= S
    A[b, :2], A[b, 2:4] = -A[a, :2], A[a, 2:4]
    return A


def bound(S, est):
    return 16 * U * S + est


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("S", [1e2, 1e4, 1e6])
def test_emulated_pair_walk(oracle, exe, kind, S):  # noqa: F811
    A, M = matrix(21, S, kind), np.ones(21, dtype=np.int32)
    ref = oracle.perm_generalized(A, M)
    for single in (True, False):
        v, kappa, *_ = emulate(exe, A, M, single)
        assert rel(v, ref) <= bound(S, kappa * U * 21), (kind, S, single)


def sparse(rows, cols):
    """Column 0 is nonzero in its last five rows only: the inner rows dominate it."""
    A = np.ascontiguousarray(I.haar_unitary(4)[:rows, :cols])
    A[:-5, 0] = 0.0
    return A


def test_emulated_column_powers(oracle, exe):  # noqa: F811
    """(With repeated columns no other column makes up for one that cancels.)"""
    A, M = sparse(19, 7), np.array([2, 2] + [1] * 17, dtype=np.int32)
    v, kappa, *_ = emulate(exe, A, M, True, False, 3)
    assert rel(v, oracle.perm_generalized(np.repeat(A, 3, axis=1), M)) <= kappa * U * 21


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [21, 22])
def test_gpu_pair_walk(oracle, kind, n):
    S, M = 1e5, np.ones(n, dtype=np.int32)
    A = matrix(n, S, kind, seed=n)
    plain = matrix(n, 1.0, kind, seed=n + 1)
    ref = oracle.perm_generalized(A, M)
    print(f"case inner rows {kind} n={n}", flush=True)
    v, info = B.perm_bbfg(A, M, with_info=True)
    assert rel(v, ref) <= bound(S, info["rel_err_est"])
    assert B.perm_bbfg_noalloc(A, M) == v
    # beside matrices whose products come from differences, replayed
    pref = oracle.perm_generalized(plain, M)
    for _ in range(4):
        out, err = B.perm_batch([(plain, M), (A, M), I.c3_item(0), (A, M)], with_err=True)
        assert rel(out[0], pref) <= err[0]
        assert rel(out[1], ref) <= bound(S, err[1]) and out[3] == out[1]


@pytest.mark.gpu
def test_gpu_column_powers(oracle):
    A, M = sparse(24, 12), np.ones(24, dtype=np.int32)
    print("case inner rows, column powers", flush=True)
    v, info = B.perm_bbfg_cols(A, M, [2] * 12, with_info=True)
    assert rel(v, oracle.perm_generalized(np.repeat(A, 2, axis=1), M)) <= info["rel_err_est"]


def minors_case(K, M, S, kind, seed=0):
    """Rows of multiplicity one first: the scaled rows are among them."""
    ones = sum(1 for x in M if x == 1)
    A = matrix(K, S, kind, seed, rows=ones)
    rng = np.random.default_rng(seed + 1000)
    more = rng.standard_normal((len(M) - ones, K)) + 1j * rng.standard_normal((len(M) - ones, K))
    return np.concatenate([A, more]), np.array(M, dtype=np.int32)


def check_minors(oracle, A, M, got, S, est=None):
    K = A.shape[1]
    for l in (2, K - 1):
        ref, absum = oracle.perm_generalized(np.delete(A, l, axis=1), M, with_abs=True)
        e = est[l] if est is not None else absum / abs(ref) * U * K
        assert rel(got[l], ref) <= 2 * bound(S, e), (l, S)


# 20 columns with one inner row; 27 with two (more than 2^18 addends)
@pytest.mark.parametrize("K,M,S", [(20, [1] * 19, 1e4), (20, [1] * 19, 1e6), (27, [1] * 18 + [4, 4], 1e6)])
@pytest.mark.parametrize("kind", KINDS)
def test_emulated_minors(oracle, minors_exe, K, M, S, kind):  # noqa: F811
    A, M = minors_case(K, M, S, kind)
    check_minors(oracle, A, M, test_minor_pairs.emulate(minors_exe, A, M, 0), S)


# two to six pairs a wavefront; the longer ones once (the oracle takes seconds)
@pytest.mark.gpu
@pytest.mark.parametrize("K,M,kind", [(K, M, kind) for K, M in ((20, [1] * 19), (24, [1] * 16 + [3, 4])) for kind in KINDS] +
                         [(27, [1] * 18 + [4, 4], "both"), (30, [1] * 18 + [5, 6], "one"),
                          (35, [1] * 18 + [8, 8], "both"), (41, [1] * 18 + [11, 11], "one")])
def test_gpu_minors(oracle, K, M, kind):
    A, M = minors_case(K, M, 1e5, kind, seed=K)
    print(f"case inner rows, minors K={K} {kind}", flush=True)
    got, est = B.perm_minors(A, M, with_err=True)
    check_minors(oracle, A, M, got, 1e5, est)
