"""The walks over pairs of columns on matrices with a value known without a sum:
zero rows and columns, infinities and NaN, all ones, the identity, derangements,
rank one, on the CPU emulation of the pair walk and on the GPU (lone sums, batch
items, minors).  Inner rows dominate every column of the identity, so it goes
without differences; the others go with them."""
import math

import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I
from tests.test_pair_walk import emulate, exe  # noqa: F401  (exe is a fixture)

TOL = 1e-10
U = 2.0 ** -53


def zero_row(n, k):
    A = np.ascontiguousarray(I.haar_unitary(3)[:n, :n])
    A[k] = 0.0
    return A


def zero_column(n, j):
    A = np.ascontiguousarray(I.haar_unitary(3)[:n, :n])
    A[:, j] = 0.0
    return A


def spoilt(n, k, j, x):
    A = np.ascontiguousarray(I.haar_unitary(3)[:n, :n])
    A[k, j] = x
    return A


def derangements(n):
    d = [1, 0]
    for k in range(2, n + 1):
        d.append((k - 1) * (d[-1] + d[-2]))
    return d[n]


def closed_forms(n):
    J = np.ones((n, n), dtype=complex)
    rng = np.random.default_rng(n)
    u, v = (np.exp(2j * np.pi * rng.random(n)) for _ in range(2))
    return [(J, math.factorial(n)), (np.eye(n, dtype=complex), 1.0), (J - np.eye(n), derangements(n)),
            (np.outer(u, v), math.factorial(n) * np.prod(u) * np.prod(v))]


@pytest.mark.parametrize("k", [0, 3, 20])
def test_emulated_zero_row(exe, k):  # noqa: F811
    """Every addend's partner cancels it: what is left is rounding, below u times the
    addends' sum for each of the n columns."""
    v, kappa, *_ = emulate(exe, zero_row(21, k), np.ones(21, dtype=np.int32))
    assert v == 0 or kappa * U * 21 >= 1


@pytest.mark.parametrize("j", [0, 11, 20])
def test_emulated_zero_column(exe, j):  # noqa: F811
    assert emulate(exe, zero_column(21, j), np.ones(21, dtype=np.int32))[0] == 0


@pytest.mark.parametrize("x", [complex(math.inf, 0), complex(0, -math.inf), complex(math.nan, 0)])
@pytest.mark.parametrize("k", [2, 20])
def test_emulated_non_finite(exe, k, x):  # noqa: F811
    v = emulate(exe, spoilt(21, k, 4, x), np.ones(21, dtype=np.int32))[0]
    assert not (math.isfinite(v.real) and math.isfinite(v.imag))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [21, 22, 24])
def test_gpu_closed_forms(n):
    M = np.ones(n, dtype=np.int32)
    for i, (A, value) in enumerate(closed_forms(n)):
        print(f"case pair edges n={n} form {i}", flush=True)
        v, info = B.perm_bbfg(A, M, with_info=True)
        assert abs(v - value) <= min(TOL, max(info["rel_err_est"], U)) * abs(value)
        w, err = B.perm_batch([(A, M)], with_err=True)
        assert abs(w[0] - value) <= min(TOL, max(err[0], U)) * abs(value)


@pytest.mark.gpu
def test_gpu_closed_forms_of_minors():
    K = 21
    M = np.ones(K - 1, dtype=np.int32)
    print("case pair edges, minors", flush=True)
    got, est = B.perm_minors(np.ones((K - 1, K), dtype=complex), M, with_err=True)
    assert (abs(got / math.factorial(K - 1) - 1) <= np.minimum(TOL, est)).all()
    eye = np.eye(K - 1, K, dtype=complex)  # only the minor without the zero column is not zero
    got = B.perm_minors(eye, M)
    assert abs(got[-1] - 1) <= 4 * U and (got[:-1] == 0).all()


@pytest.mark.gpu
def test_gpu_zero_and_non_finite():
    n = 21
    M = np.ones(n, dtype=np.int32)
    plain = np.ascontiguousarray(I.haar_unitary(3)[:n, :n])
    want = B.perm_batch([(plain, M)])[0]
    inf, nan = math.inf, math.nan
    bad = [spoilt(n, k, 4, x) for k in (2, 20) for x in (complex(inf, 0), complex(0, -inf), complex(nan, 0))]
    print("case pair edges, zero and non-finite", flush=True)
    for k in (0, 3, 20):
        v, info = B.perm_bbfg(zero_row(n, k), M, with_info=True)
        assert v == 0 or info["rel_err_est"] >= 1
        assert B.perm_bbfg(zero_column(n, k), M) == 0
    for A in bad:
        v = B.perm_bbfg(A, M)
        assert not (math.isfinite(v.real) and math.isfinite(v.imag))
        m = B.perm_minors(A[1:], M[1:])
        # the minor without the spoilt column is what it is without it
        clean = A[1:].copy()
        clean[:, 4] = 0.0
        ref = B.perm_minors(clean, M[1:])[4]
        assert not np.isfinite(np.delete(m, 4)).any()
        assert abs(m[4] - ref) <= 1e-12 * abs(ref)
    # items beside them keep their bits
    out = B.perm_batch([(plain, M), (bad[0], M), (plain, M), (bad[5], M), (zero_column(n, 4), M)])
    assert out[0] == want and out[2] == want and out[4] == 0
    assert not np.isfinite(out[[1, 3]]).any()
