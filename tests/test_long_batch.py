"""A batch whose pair-walk tables exceed their bound runs as several launches over
one buffer: 8192 items of 24 photons (2.4 GB of tables) over eight matrices, so
that equal items stand in every launch.  Equal items give equal bits, those of
the item alone; the device memory taken stays near the bound; calls repeat (the
captured sequence holds all launches)."""
import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_tables_within_their_bound(oracle):
    import torch
    n, count, distinct = 24, 8192, 8
    A = np.stack([I.haar_unitary(40 + i)[:n, :n] for i in range(distinct)])
    At = torch.from_numpy(np.ascontiguousarray(A.ravel())).cuda()
    ones = np.ones(n, dtype=np.int32)
    alone = np.array([B.perm_batch([(A[i], ones)])[0] for i in range(distinct)])
    which = np.arange(count) % distinct
    args = (At, which.astype(np.int64) * n * n, np.full(count, n), np.tile(ones, count), np.arange(count) * n,
            np.full(count, n))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    print("case long batch", flush=True)
    for rep in range(3):
        B.perm_bbfg(A[0][:6, :6])
        out, err = B.perm_batch_packed(*args, with_err=True)
        assert np.array_equal(out, alone[which])
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken < 1.75 * 2 ** 30
    ref = oracle.perm_generalized(A[3], ones)
    assert abs(out[3] - ref) <= min(1e-10, err[3]) * abs(ref)
