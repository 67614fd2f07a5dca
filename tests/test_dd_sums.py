"""Sums that the kernels hold in double-double, in their own code compiled for the
host: where plain FP64 loses the small terms beside large ones that cancel, the
exact sum comes out."""
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2309_07027_amd" / "csrc"


def run(tmp_path, body):
    src = tmp_path / "sums.cpp"
    src.write_text('#include <cstdio>\n#include "pair_core.hpp"\nusing namespace bbfg;\nint main()\n{\n' + body + "\n}\n")
    exe = tmp_path / "sums"
    subprocess.run(["g++", "-O1", "-std=c++17", "-ffp-contract=off", "-Wno-unknown-pragmas", f"-I{CSRC}",
                    f"-I{ROOT / 'include'}", str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, check=True)
    return [float.fromhex(x) for x in p.stdout.split()]


def test_a_units_sum_over_its_wavefronts(tmp_path):
    """Large values of both signs, and 1 + v / 1024 in wavefront v; weights of two
    wavefronts, 3 and -5."""
    hi_r, hi_i, sa = run(tmp_path, """
    double r[kPairWaves], i[kPairWaves], m[kPairWaves], w[kPairWaves];
    for (int v = 0; v < kPairWaves; ++v) {
        r[v] = 1.0 + v / 1024.0;
        i[v] = -r[v];
        m[v] = 1.0;
        w[v] = v == 4 ? 3.0 : v == 7 ? -5.0 : 1.0;
    }
    r[1] = 0x1p70;
    r[6] = -0x1p70;
    i[2] = -0x1p66;
    i[15] = 0x1p66;
    ddv sr, si;
    double sa;
    pair_join([&](int v, double& a, double& b, double& c, double& d) { a = r[v]; b = i[v]; c = m[v]; d = w[v]; },
              r[0], i[0], m[0], w[0], sr, si, sa);
    std::printf("%a %a %a\\n", sr.hi + sr.lo, si.hi + si.lo, sa);
    return 0;""")
    value = [1 + v / 1024 for v in range(16)]
    assert hi_r == -15 * sum(x for v, x in enumerate(value) if v not in (1, 6))
    assert hi_i == 15 * sum(x for v, x in enumerate(value) if v not in (2, 15))
    assert sa == 15 * 16


def test_a_running_sum(tmp_path):
    """What the first steps of a sample add their threads' sums with."""
    total, = run(tmp_path, """
    ddv s = {0.0, 0.0};
    for (int i = 0; i < 64; ++i) dd_gather(s, i == 5 ? 0x1p60 : i == 50 ? -0x1p60 : 1.0 + i / 4096.0);
    std::printf("%a\\n", s.hi + s.lo);
    return 0;""")
    assert total == sum(1 + i / 4096 for i in range(64) if i not in (5, 50))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2, 9, 10, 11, 12, 14])
def test_estimate_of_the_first_steps_of_a_sample(n):
    """n photons in one mode: step k's minors are all (k - 1)!, whatever the order, so
    the estimate is the sum over the steps of dw / w with dw = e (2 sqrt(w) + e),
    sqrt(w) = k!, e = k! kappa u (k - 1 + sqrt(Q)), Q the Gray positions a thread
    walks from one seed: one up to ten columns, doubling with each further one."""
    from math import comb, factorial

    import numpy as np

    from paper_2309_07027_amd import binding as B
    u = 2.0 ** -53
    want = 0.0
    for k in range(2, n + 1):
        q = k - 1  # photons of a minor
        kappa = sum(comb(q - 1, d) * abs(q - 2 * d) ** q for d in range(q)) / 2 ** (q - 1) / factorial(q)
        e = kappa * u * (q + 2.0 ** (max(0, k - 10) / 2))
        want += e * (2 + e)
    print(f"case early estimate n={n}", flush=True)
    got, info = B.bs_sample(np.ones((1, 1), dtype=complex), [n], 3, 0.0, 1, with_info=True)
    assert (got == n).all()
    assert abs(info["rel_err_est"] / want - 1) < 1e-9
