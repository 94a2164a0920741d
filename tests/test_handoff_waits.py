"""The kernels whose workgroups hand their results to the one that arrives
last, in the assembly the build flags give: before the barrier that stands in
front of the write-back of the L2, every wave waits for its own stores (the
barrier itself waits for LDS only, and the write-back covers what has reached
the L2).  CPU only: the kernels are compiled, not run."""
import os
import re
import subprocess

import pytest

from paper_2102_05297_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "sweep.s")
    subprocess.run([build.hipcc(), *build.COMMON, *build.SOURCES["sweep.hip"], "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, "sweep.hip"), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    return {name: body.splitlines() for name, body in
            re.findall(r"^(_ZN3cgs\w+):\s.*?\n(.*?)^\.Lfunc_end", text, re.M | re.S)}


@pytest.mark.parametrize("kernel", ["small_step", "batch_small", "nb_stepILi2E", "nb_stepILi8E", "nb_stepILi16E"])
def test_stores_are_waited_for_before_the_handoff(kernels, kernel):
    (lines,) = [b for n, b in kernels.items() if kernel in n]
    back = [i for i, l in enumerate(lines) if "buffer_wbl2" in l]
    assert back, "the kernel has no handoff"
    for b in back:
        barrier = max(i for i in range(b) if "s_barrier" in lines[i])
        store = max(i for i in range(barrier) if re.search(r"\b(global|flat)_(store|atomic)", lines[i]))
        waits = [l for l in lines[store:barrier] if "s_waitcnt" in l and "vmcnt(0)" in l]
        assert waits, f"no wait between the store and the barrier: {lines[store].strip()}"
