"""The server's device time counts the first steps of samples also where they run in
a step beside other samples' walks, as its flops do: samples of 14 photons (first
steps only) submitted while jobs of 27 photons run in both halves take at least
half of what they take alone on top of those jobs' time."""
import time

import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

pytestmark = pytest.mark.gpu


def walk_ms(long_jobs, short_jobs):
    U = I.haar_unitary(5, 40)
    occ = lambda n: np.array([1] * n + [0] * (40 - n), dtype=np.int32)  # noqa: E731
    with B.Server() as srv:
        for i in range(long_jobs):
            srv.submit(U, occ(27), 256, 0.0, i)
        if long_jobs and short_jobs:
            time.sleep(0.015)  # of the 45 ms that the long jobs take: they are at their walks
        for i in range(short_jobs):
            srv.submit(U, occ(14), 4096, 0.0, 100 + i)
        srv.drain()
        return srv.stats()["walk_ms"]


def test_first_steps_beside_walks_are_timed():
    walk_ms(2, 2)  # plans, tables and clocks come up
    print("case server times", flush=True)
    alone = walk_ms(0, 6)
    assert alone > 1.0
    assert walk_ms(2, 6) >= 0.95 * walk_ms(2, 0) + 0.5 * alone
