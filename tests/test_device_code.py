"""CPU test: what the compiler makes of the linear layers' kernels (assembly of gfx950, built here, nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_2403_02310_amd import build


@pytest.fixture(scope="module")
def linear_assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "linear.s")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--offload-device-only", "-S", "-o", out,
                    os.path.join(build.CSRC, "linear_kernels.hip")], check=True, capture_output=True)
    return open(out).read()


def test_output_strips_are_ordered_between_the_lanes_of_a_wavefront(linear_assembly):
    """The way out of a large tile turns 32 tokens at a time in LDS: lanes read what other lanes of the wavefront wrote.  The
    source states the order (a wavefront barrier, for which no instruction is issued) and the compiler keeps it: behind
    the key loop no LDS read follows LDS writes without one in between."""
    bodies = re.findall(r"^(\S*linear_phased_kernel\S*):.*?\n(.*?)^\.Lfunc_end", linear_assembly, re.S | re.M)
    assert len(bodies) == 21
    for name, body in bodies:
        lines = [l.strip() for l in body.splitlines()]
        start = max(i for i, l in enumerate(lines) if l.startswith("s_barrier"))
        written, reads = False, 0
        for l in lines[start:]:
            if "wave barrier" in l:
                written = False
            elif l.startswith("ds_write"):
                written = True
            elif l.startswith("ds_read"):
                assert not written, (name, l)
                reads += 1
        assert reads >= 12, name
