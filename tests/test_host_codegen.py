"""Order of the completion atomics in the step kernels as compiled for gfx950
(hipcc only, no GPU): a workgroup's arrival may be counted only once its
speed and error atomics have been performed, because the last arrival reads
what they left.  An atomic whose result is unused is not waited for by
itself, and a result compared with a value that it cannot have is unused."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1705_00614_amd import build

KERNELS = {
    "batch_f32": "k_batch_step<float, 32, 32, 512, 0>(swe::BatchArgs<float>)",
    "batch_f64": "k_batch_step<double, 16, 16, 512, 0>(swe::BatchArgs<double>)",
    "step_f32": "k_step<float, 32, 32, 512, 0, 0>(swe::Args<float>)",
    "step_f64": "k_step<double, 16, 16, 512, 0, 0>(swe::Args<double>)",
    "step_grids": "k_step_grids<float, 32, 32, 512, 0>(const swe::Args<float>*, swe::GridShares)",
    "nest_close": "k_nest_close<float>(swe::Args<float>, swe::NestArgs<float>, const int*, const int*, int, int, int)",
}
CONTRIBUTION = re.compile(r"\s(global|flat)_atomic_(umax|cmpswap)\S*\s")   # speeds and errors
ARRIVAL = re.compile(r"\s(global|flat)_atomic_add_x2\s")                   # the group's 64-bit arrival word


def _compile(tmp_path, kernel):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text('#include "%s"\ntemplate __global__ void swe::%s;\n'
                   % (os.path.join(build.CSRC, "swe_nest.hpp"), kernel))
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    res = subprocess.run(["hipcc"] + flags + ["--cuda-device-only", "-S", "-o", str(asm), str(src)], check=True,
                         capture_output=True, text=True)
    return [line.split(";")[0] for line in asm.read_text().split("\n")], res.stderr


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("name", sorted(KERNELS))
def test_contributions_are_waited_for_before_the_arrival(tmp_path, name):
    lines, _ = _compile(tmp_path, KERNELS[name])
    arrivals = [k for k, line in enumerate(lines) if ARRIVAL.search(line)]
    contributions = [k for k, line in enumerate(lines) if CONTRIBUTION.search(line)]
    assert len(arrivals) == 1 and contributions, (arrivals, contributions)
    assert max(contributions) < arrivals[0]
    # every path from a contribution to the arrival passes the last barrier
    # before the arrival: either a drain stands behind that barrier, or the
    # contribution returns a value (sc0) that is waited for before it
    barrier = max(k for k in range(arrivals[0]) if lines[k].strip() == "s_barrier")

    def drained(first, end):
        return any("s_waitcnt" in line and "vmcnt(0)" in line for line in lines[first:end])

    for k in contributions:
        assert drained(barrier, arrivals[0]) or (" sc0" in lines[k] and drained(k, barrier)), lines[k]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("tile", ["double, 16, 16, 512", "double, 32, 16, 512", "float, 64, 16, 512", "float, 16, 16, 256"])
def test_kernels_ask_for_waves_that_fit(tmp_path, tile):
    """The waves per SIMD a step kernel is compiled for fit its tile's LDS."""
    _, said = _compile(tmp_path, "k_step<%s, 0, 0>(swe::Args<%s>)" % (tile, tile.split(",")[0]))
    assert "failed to meet occupancy" not in said, said
