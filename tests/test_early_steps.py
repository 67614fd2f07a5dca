"""The first steps of a sample run in one launch (up to 14), later ones in one
each: samples equal to the oracle's at photon counts on both sides of that line
and of the eight signs a thread holds, with repeated rows (few modes), a doubled
interferometer and input loss.  Samples are compared exactly: both sides use the
same uniforms, and the weights agree to far better than the gaps between them."""
import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1, 5), (2, 3), (9, 6), (10, 12), (11, 40), (14, 16), (15, 16), (16, 20)])
def test_samples_equal_the_oracle(oracle, n, m):
    U = I.haar_from_rng(np.random.default_rng(100 + n), m)
    occ = np.zeros(m, dtype=np.int32)
    for i in range(n):
        occ[i % m] += 1
    print(f"case early steps n={n} m={m}", flush=True)
    got, info = B.bs_sample(U, occ, 5, 0.0, n, with_info=True)
    assert np.array_equal(got, oracle.cc_sample(U, occ, 5, 0.0, n))
    assert n == 1 or 0 < info["rel_err_est"] < 1e-6
    assert np.array_equal(B.bs_sample(U, occ, 3, 0.4, n), oracle.cc_sample(U, occ, 3, 0.4, n))
    assert np.array_equal(B.bs_sample_extracted(U, occ, 6, 0.3, n), oracle.cc_sample_extracted(U, occ, 6, 0.3, n))


def test_addends_are_counted_as_for_single_steps():
    """info's addend count: k minors of prod (M'_k + 1) addends per step."""
    U = I.haar_from_rng(np.random.default_rng(3), 4)
    occ = np.array([3, 3, 0, 0], dtype=np.int32)
    print("case early steps addends", flush=True)
    got, info = B.bs_sample(U, occ, 1, 0.0, 5, with_info=True)
    assert got.sum() == 6
    # every prefix of five photons on four modes has between 2 and 2^4 addends
    assert sum(k for k in range(2, 7)) <= info["n_addends"] <= sum(k * 2 ** (k - 2) for k in range(2, 7))
