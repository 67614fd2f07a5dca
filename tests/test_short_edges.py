"""Where the one-launch permanent ends: unit counts on both sides of 256 (one or
four wavefronts a work group) and of 2048 (the general sequence beyond), each
asserted, with the bits of the general sequence; and calls of several threads on
streams of their own."""
import threading

import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu

# multiplicities without four binary digits, which the pair walk would take
CASES = {
    252: [1, 2, 2, 3, 3, 3, 3, 3, 6],
    258: [3, 3, 3, 3, 6, 6, 6],
    2025: [1, 1, 1, 2, 2, 2, 2, 2, 2, 3, 4, 4, 6],
    2048: [1, 1] + [3] * 10,
    2049: [1, 1, 2, 2, 2, 2, 2, 2, 2, 3, 3, 4, 5],
    2051: [1, 2, 2, 2, 2, 2, 2, 2, 2, 3, 3, 3, 4],
}


def matrix(M, seed=23):
    return np.ascontiguousarray(I.haar_unitary(seed)[:len(M), :sum(M)]), np.array(M, dtype=np.int32)


@pytest.mark.parametrize("units", sorted(CASES))
def test_unit_counts(oracle, units):
    A, M = matrix(CASES[units])
    print(f"case short edges {units} units", flush=True)
    ref, rinfo = B.perm_bbfg_noalloc(A, M, with_info=True)
    assert rinfo["n_units"] == units
    for _ in range(3):
        got, info = B.perm_bbfg(A, M, with_info=True)
        assert got == ref and info["n_units"] == units
        assert info["kappa"] == rinfo["kappa"] and info["rel_err_est"] == rinfo["rel_err_est"]
    assert abs(got - oracle.perm_generalized(A, M)) <= info["rel_err_est"] * abs(got)


def test_threads_on_streams_of_their_own():
    import torch
    cases = [matrix(M) for M in ([1] * 20, [1] * 10, CASES[258], [1, 2, 1])]
    refs = [B.perm_bbfg_noalloc(A, M) for A, M in cases]
    print("case short edges, threads", flush=True)
    wrong = []

    def work(i):
        stream = torch.cuda.Stream()
        B.set_stream(stream)
        try:
            for rep in range(40):
                j = (i + rep) % len(cases)
                if B.perm_bbfg(*cases[j]) != refs[j]:
                    wrong.append((i, rep, j))
        finally:
            B.set_stream(None)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert wrong == []
