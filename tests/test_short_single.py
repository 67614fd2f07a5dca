"""Short single permanents in one launch against the general launch sequence
(perm_bbfg_noalloc runs the same plan through it): the same bits, at one unit,
on both sides of 256 units (one or four wavefronts a work group) and of the
largest unit count, at 24, 32 and 33 columns, with few and many kept rows, rows
of multiplicity zero, host and device matrices, repeated calls and another
stream; and against the oracle."""
import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = {
    "one_unit": [1, 2, 1],
    "one_row": [9],
    "one_column": [1],
    "two_units": [1] * 10,
    "units_256": [1] * 17,
    "units_257": [1] * 13 + [2, 2, 3],
    "units_1024": [1] * 20,
    "bunched_24": [4, 4, 5, 3, 2, 6],
    "columns_32": [3, 5, 4, 6, 2, 7, 5],
    "columns_33": [3, 5, 4, 6, 2, 7, 6],
    "zero_rows": [0, 2, 0, 3, 1, 0, 1, 1, 1, 1],
}


def matrix(M):
    return np.ascontiguousarray(I.haar_unitary(21)[:len(M), :sum(M)]), np.array(M, dtype=np.int32)


@pytest.mark.parametrize("name", sorted(CASES))
def test_same_bits_as_the_general_sequence(oracle, name):
    import torch
    A, M = matrix(CASES[name])
    print(f"case short single {name}", flush=True)
    ref, rinfo = B.perm_bbfg_noalloc(A, M, with_info=True)
    B.perm_bbfg(A, M)  # brings the Gray table to the device
    At = torch.from_numpy(A).cuda()
    for X in (A, At, A):
        got, info = B.perm_bbfg(X, M, with_info=True)
        assert got == ref and info["kappa"] == rinfo["kappa"] and info["rel_err_est"] == rinfo["rel_err_est"]
        assert info["n_units"] == rinfo["n_units"]
    assert abs(got - oracle.perm_generalized(A, M)) <= max(1e-10 * abs(got), rinfo["rel_err_est"] * abs(got))
    r, rr = B.perm_ryser(At, M, with_info=True)
    assert abs(r - ref) <= (rr["rel_err_est"] + 1e-12) * abs(ref)


def test_calls_in_turn_on_two_streams():
    """The counters of finished work groups are back at zero after every launch."""
    import torch
    cases = [matrix(CASES[c]) for c in ("units_1024", "two_units", "units_257", "one_unit")]
    refs = [B.perm_bbfg_noalloc(A, M) for A, M in cases]
    print("case short single, two streams", flush=True)
    stream = torch.cuda.Stream()
    try:
        for rep in range(6):
            B.set_stream(stream if rep % 2 else None)
            for (A, M), ref in zip(cases, refs):
                assert B.perm_bbfg(A, M) == ref
    finally:
        B.set_stream(None)
