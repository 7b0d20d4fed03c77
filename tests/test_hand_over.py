"""What the values that pass between the blocks of one launch are compiled to: read-modify-writes on both sides.  (A
read-modify-write the compiler can see through, such as the addition of a constant zero, becomes a plain load.)"""
import os
import re
import subprocess

import pytest

from paper_2403_04206_amd import buildlib

PROBE = """
#include "grawa_scores.h"
extern "C" __global__ void probe_hand_over(double *p, double v) { hand_over(p + threadIdx.x, v); }
extern "C" __global__ void probe_take_over(double *p, double *out) { out[threadIdx.x] = take_over(p + threadIdx.x); }
"""


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    try:
        hipcc = buildlib.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("asm")
    src, asm = str(d / "probe.hip"), str(d / "probe.s")
    with open(src, "w") as f:
        f.write(PROBE)
    cmd = [hipcc] + buildlib.HIPCC_FLAGS + ["-w", "-I", os.path.join(buildlib.ROOT, "include"), "-I", buildlib.CSRC,
                                            "--offload-device-only", "-S", src, "-o", asm]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    text = open(asm).read()
    return {n: re.search(r"^%s:(.*?)s_endpgm" % n, text, re.S | re.M).group(1) for n in ("probe_hand_over", "probe_take_over")}


def test_hand_over_is_an_exchange_that_is_waited_for(kernels):
    assert re.search(r"global_atomic_swap_x2 .*sc0\s*\n(.*\n)*?\s*s_waitcnt vmcnt\(0\)", kernels["probe_hand_over"])
    assert not re.search(r"global_store|flat_store", kernels["probe_hand_over"])


def test_take_over_is_a_read_modify_write(kernels):
    assert re.search(r"global_atomic_add_x2 .*sc0", kernels["probe_take_over"])
    assert not re.search(r"global_load|flat_load", kernels["probe_take_over"])
