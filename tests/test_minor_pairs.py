"""The leave-one-column-out walk over pairs of columns against the oracle: on the
CPU its per-lane code on the planner's split with bounds-checked reads
(tests/emu/minor_pairs_emu.cpp), on the GPU through perm_minors.  Column counts
on both sides of each step in the pairs per wavefront, odd and even, equal and
unequal shares, columns that leave a wavefront without any, rows of multiplicity
above one.  The bound
is the FP64 path's (1e-10 relative to the oracle where its kappa is at most 1e6,
and always the reported estimate)."""
import os
import subprocess
from pathlib import Path

import numpy as np
import pytest

from paper_2309_07027_amd import binding as B
from paper_2309_07027_amd import inputs as I

HERE = Path(__file__).resolve().parent
ROOT = HERE.parent
CSRC = ROOT / "paper_2309_07027_amd" / "csrc"
TOL = 1e-10


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("minor_emu") / "minor_pairs_emu"
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-ffp-contract=off", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-Wall", "-Wno-unknown-pragmas",
                    f"-I{CSRC}", f"-I{ROOT / 'include'}", str(HERE / "emu" / "minor_pairs_emu.cpp"),
                    str(CSRC / "plan.cpp"), "-o", str(out)], check=True)
    return out


def emulate(exe, A, M, l_batch, slots=512):
    text = "\n".join([f"{A.shape[0]} {A.shape[1]} {slots} {l_batch}", " ".join(map(str, M)),
                      " ".join(f"{float(x.real).hex()} {float(x.imag).hex()}" for x in A.ravel())])
    p = subprocess.run([str(exe)], input=text + "\n", capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert p.returncode == 0, p.stderr[-2000:]
    if p.stdout.startswith("general"):
        return None
    v = [float.fromhex(x) for x in p.stdout.split()]
    return np.array([complex(a, b) for a, b in zip(v[0::2], v[1::2])])


def multiplicities(K, addends):
    """K - 1 photons with about `addends` sign patterns: single rows, and a few
    heavily occupied ones for the rest."""
    ones = max(3, int(np.log2(addends)) - 3)
    if ones >= K - 1:
        return [1] * (K - 1)
    left = K - 1 - ones
    a = (left + 1) // 2
    return [1] * ones + [a] + ([left - a] if left > a else [])


def case(K, addends, seed=5):
    M = multiplicities(K, addends)
    return np.ascontiguousarray(I.haar_unitary(seed)[:len(M), :K]), np.array(M, dtype=np.int32)


def check(oracle, A, M, got, est=None, every=1):
    for l in range(0, A.shape[1], every):
        ref, absum = oracle.perm_generalized(np.delete(A, l, axis=1), M, with_abs=True)
        e = abs(got[l] - ref) / abs(ref)
        kappa = absum / abs(ref)
        assert e <= (TOL if kappa <= 1e6 else kappa * 2.0 ** -53 * 200), (l, e, kappa)
        if est is not None:
            assert e <= est[l], (l, e, est[l])


@pytest.mark.parametrize("K", [10, 15, 16, 17, 24, 25, 27, 30, 32, 33, 38, 40, 41, 48])
def test_emulation_matches_oracle(oracle, exe, K):
    A, M = case(K, 2 ** 14)
    got = emulate(exe, A, M, 64)
    assert got is not None
    check(oracle, A, M, got, every=5)


def test_planner_leaves_short_sums_and_bunched_rows_to_the_other_walk(exe):
    assert emulate(exe, *case(8, 2 ** 20), 64) is None                                  # too few columns
    assert emulate(exe, *case(16, 2 ** 16), 0) is None                                  # alone, 2^14 addends
    A = np.ascontiguousarray(I.haar_unitary(1)[:8, :17])
    assert emulate(exe, A, np.array([2] * 8, dtype=np.int32), 64) is None               # no row of multiplicity one


@pytest.mark.parametrize("K", [25, 27, 32])
def test_emulation_of_two_inner_digits(oracle, exe, K):
    """25 to 32 columns and more than 2^18 addends: two inner digits.  A few
    minors, those at both ends of a wavefront's columns among them."""
    A, M = case(K, 2 ** 19)
    got = emulate(exe, A, M, 512)
    check(oracle, A, M, got, every=8)


@pytest.mark.gpu
@pytest.mark.parametrize("K", [17, 20, 24, 25, 27, 29, 32, 33, 36, 40, 41, 48])
def test_gpu_matches_oracle(oracle, K):
    A, M = case(K, 2 ** 19)
    print(f"case minors over pairs K={K} M={M.tolist()}", flush=True)
    got, est = B.perm_minors(A, M, with_err=True)
    check(oracle, A, M, got, est, every=13)


@pytest.mark.gpu
@pytest.mark.parametrize("K", [22, 33])
def test_gpu_estimate_with_a_zero_column(K):
    """Only the minor that drops the zero column is not zero; its estimate is finite."""
    A, M = case(K, 2 ** 21)
    A[:, 5] = 0.0
    print(f"case minors over pairs, zero column K={K}", flush=True)
    got, est = B.perm_minors(A, M, with_err=True)
    assert np.isfinite(est[5]) and 0.0 < est[5] < 1e-6
    assert all(got[l] == 0 for l in range(K) if l != 5)


@pytest.mark.gpu
def test_gpu_samples_equal_the_oracle_sampler(oracle):
    """A step of a sampling call mixes both walks and several column counts."""
    U = I.haar_from_rng(np.random.default_rng(77), 20)
    occ = np.array([1] * 14 + [0] * 6, dtype=np.int32)
    print("case sampler over both minors walks", flush=True)
    assert np.array_equal(B.bs_sample(U, occ, 6, 0.0, 13), oracle.cc_sample(U, occ, 6, 0.0, 13))
