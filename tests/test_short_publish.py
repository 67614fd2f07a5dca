"""The one-launch permanent publishes every wavefront's partial record before its
work group is counted.  A work group's barrier on this target waits for no
vector store, and the release before the count is executed by one wavefront, so
each storing wavefront has to wait for its own stores.  Read off the compiled
kernels, on the CPU: between the last store of a partial and the barrier that
precedes the count stands a wait for all outstanding vector memory operations."""
import re
import subprocess
from pathlib import Path

import pytest

from paper_2309_07027_amd import build as bld


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("short") / "short.s"
    subprocess.run([bld.HIPCC, *bld.COMMON, *bld.HIP_FLAGS, "-w", "-S", "--offload-device-only",
                    str(bld.CSRC / "walk_short.hip"), "-o", str(out)], check=True, timeout=600)
    text = out.read_text()
    found = re.findall(r"^(_ZN4bbfg\S*walk_short_kernel\S*):\s*;.*?\n(.*?)^\.Lfunc_end", text, re.S | re.M)
    assert len(found) == 32
    return dict(found)


def test_a_wavefront_waits_for_its_partial_before_the_count(kernels):
    for name, body in kernels.items():
        lines = [x.strip() for x in body.splitlines()]
        count = next(i for i, x in enumerate(lines) if x.startswith("global_atomic_add"))
        barrier = max(i for i in range(count) if lines[i].startswith("s_barrier"))
        store = max(i for i in range(barrier) if lines[i].startswith("global_store_dwordx2"))
        assert any(re.match(r"s_waitcnt.*vmcnt\(0\)", x) for x in lines[store:barrier]), name
