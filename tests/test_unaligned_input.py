"""Device matrices aligned to a double but not to a complex element: the entry
points take pointers to pairs of doubles, so half of all addresses are such.
Same bits as for the aligned copy: one-launch permanents of one unit and of many,
the pair walk and the minors."""
import ctypes

import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu


def call(f, ptr, A, M, results):
    out = np.zeros(results, dtype=np.complex128)
    m = np.ascontiguousarray(M, dtype=np.int32)
    B._check(f(ctypes.c_void_p(ptr), A.shape[0], m.ctypes.data_as(B._PI32), A.shape[1],
               ctypes.c_void_p(out.ctypes.data), None))
    return out


@pytest.mark.parametrize("n", [3, 8, 17, 20, 22])
def test_same_bits_as_aligned(n):
    import torch
    A = np.ascontiguousarray(I.haar_unitary(31)[:n, :n])
    flat = torch.from_numpy(A.view(np.float64).ravel()).cuda()
    shifted = torch.zeros(flat.numel() + 1, dtype=torch.float64, device="cuda")
    shifted[1:] = flat
    torch.cuda.synchronize()
    assert flat.data_ptr() % 16 == 0
    M = np.ones(n, dtype=np.int32)
    L = B.lib()
    print(f"case unaligned input n={n}", flush=True)
    for f, m, results in ((L.perm_bbfg, M, 1), (L.perm_ryser, M, 1), (L.perm_minors, M[1:], n)):
        X = A if results == 1 else A[1:]
        skip = 0 if results == 1 else 16 * n
        for _ in range(2):  # the second call finds the Gray table resident
            want = call(f, flat.data_ptr() + skip, X, m, results)
            got = call(f, shifted.data_ptr() + 8 + skip, X, m, results)
            assert np.array_equal(want, got)
