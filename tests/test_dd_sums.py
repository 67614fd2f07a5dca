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
