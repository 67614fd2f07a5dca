"""The pair walk (sums of more than 2^19 addends) against the oracle.

On the CPU its per-lane code runs on the planner's split with bounds-checked
reads (tests/emu/pair_emu.cpp): odd and even column counts, rows of multiplicity
above one on lane, mid and high digits, lane groups that leave lanes idle, the
Ryser formula and column powers, alone and batched.  On the GPU every entry
point that reaches it.  The bound is the FP64 path's, a relative error of 1e-10
and, always, the reported estimate kappa u (n + sqrt(Q)).
"""
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

# (multiplicities, Ryser): just above 2^19 addends
CASES = {
    "distinct_odd": ([1] * 21, False),
    "distinct_even": ([1] * 22, False),
    "doubles": ([1] * 13 + [2] * 5, False),
    "triples_fours": ([1] * 9 + [3, 3, 4, 2, 2, 2], False),
    "few_binary_digits": ([1] * 6 + [2, 3, 4, 5, 6, 7], False),
    "ryser": ([1] * 16 + [2, 2, 2], True),
}


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("pair_emu") / "pair_emu"
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-ffp-contract=off", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-fno-omit-frame-pointer", "-Wall", "-Wno-unknown-pragmas",
                    f"-I{CSRC}", f"-I{ROOT / 'include'}", str(HERE / "emu" / "pair_emu.cpp"), str(CSRC / "plan.cpp"),
                    "-o", str(out)], check=True)
    return out


def emulate(exe, A, M, single=True, ryser=False, power=0):
    A = np.ascontiguousarray(A, dtype=np.complex128)
    text = "\n".join([f"{A.shape[0]} {A.shape[1]} {int(single)} {int(ryser)} {power}", " ".join(map(str, M)),
                      " ".join(f"{float(x.real).hex()} {float(x.imag).hex()}" for x in A.ravel())])
    p = subprocess.run([str(exe)], input=text + "\n", capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert p.returncode == 0, p.stderr[-2000:]
    if p.stdout.startswith("general"):
        return None
    re_, im_, kappa, units, mid = p.stdout.split()
    return complex(float.fromhex(re_), float.fromhex(im_)), float.fromhex(kappa), int(units), int(mid)


def matrix(M, n=None, seed=11):
    n = n or sum(M)
    u = I.haar_unitary(seed)
    return np.ascontiguousarray(u[:len(M), :n]), np.array(M, dtype=np.int32)


def rel(a, b):
    return abs(a - b) / abs(b)


@pytest.mark.parametrize("name", sorted(CASES))
def test_emulation_matches_oracle(oracle, exe, name):
    M, ryser = CASES[name]
    A, M = matrix(M)
    ref, absum = oracle.perm_generalized(A, M, with_abs=True)
    for single in (True, False):
        v, kappa, units, mid = emulate(exe, A, M, single, ryser)
        assert rel(v, ref) <= (TOL if not ryser else kappa * 2.0 ** -53 * 200), (name, single, units, mid)
        if not ryser:  # kappa is the oracle's sum of |re| + |im| over |perm|, between 1 and sqrt(2) of its moduli
            assert 1.0 <= kappa / (absum / abs(ref)) <= 1.4143


def test_emulation_of_column_powers(oracle, exe):
    M = [1] * 17 + [2, 2]
    A, M = matrix(M, 7)
    v, kappa, *_ = emulate(exe, A, M, True, False, 3)
    assert rel(v, oracle.perm_generalized(np.repeat(A, 3, axis=1), M)) <= TOL


def test_planner_leaves_short_and_bunched_sums_to_the_general_walk(exe):
    assert emulate(exe, *matrix([1] * 20)) is None          # 2^19 addends
    assert emulate(exe, *matrix([4] * 10)) is None          # no binary digits


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(CASES))
def test_gpu_matches_oracle(oracle, name):
    M, ryser = CASES[name]
    A, M = matrix(M)
    ref = oracle.perm_generalized(A, M)
    print(f"case pair walk {name}", flush=True)
    f = B.perm_ryser if ryser else B.perm_bbfg
    v, info = f(A, M, with_info=True)
    assert rel(v, ref) <= info["rel_err_est"]
    assert ryser or rel(v, ref) <= TOL
    # in a mix of short sums, repeated: same bits alone, mixed and replayed
    small = [I.c3_item(i) for i in range(5)]
    prec = B.BBFG_RYSER if ryser else B.BBFG_FP64
    alone = B.perm_batch([(A, M)], precision=prec)[0]
    for _ in range(4):
        B.perm_bbfg(*small[0])
        out, err = B.perm_batch(small[:2] + [(A, M), (A[::-1].copy(), M[::-1].copy())] + small[2:], precision=prec,
                                with_err=True)
        assert out[2] == alone
        assert rel(out[3], ref) <= max(err[3], 1e-15) and rel(out[2], ref) <= max(err[2], 1e-15)
    if not ryser:
        assert B.perm_bbfg_noalloc(A, M) == v


@pytest.mark.gpu
@pytest.mark.parametrize("power", [2, 3, 4])
def test_gpu_column_powers(oracle, power):
    C = {2: 12, 3: 8, 4: 6}[power]
    n = C * power
    M = [1] * n
    A, M = matrix(M, C)
    print(f"case pair walk column power {power}", flush=True)
    v, info = B.perm_bbfg_cols(A, M, [power] * C, with_info=True)
    assert info["n_addends"] == 2 ** 23
    assert rel(v, oracle.perm_generalized(np.repeat(A, power, axis=1), M)) <= min(TOL, info["rel_err_est"])


@pytest.mark.gpu
def test_gpu_largest_column_count(oracle):
    """n = 48: 24 pairs, the LDS of a whole compute unit."""
    M = [1] * 12 + [12, 12, 12]
    A, M = matrix(M)
    print("case pair walk n=48", flush=True)
    v, info = B.perm_bbfg(A, M, with_info=True)
    assert rel(v, oracle.perm_generalized(A, M)) <= info["rel_err_est"]
