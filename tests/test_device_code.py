"""What the compiler makes of device code where a property of the source has to hold and no
run can show it (the library's own sources, compiled here; no GPU needed)."""

import os
import re
import subprocess

from paper_2208_12569_amd import build


def _ir(src, tmp_path):
    out = str(tmp_path / "device.ll")
    subprocess.check_call([build.HIPCC, "--offload-arch=gfx950", "--offload-device-only", "-O1", "-std=c++17", "-w", "-S",
                           "-emit-llvm", "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(build.CSRC, src), "-o", out])
    with open(out) as fh:
        return fh.read()


def test_lanes_exchange_lds_between_fences(tmp_path):
    """A wave barrier orders scheduling only: where a wave's lanes read what other lanes
    wrote to LDS, a release fence stands before it and an acquire fence after it."""
    ir = _ir("prep.hip", tmp_path).splitlines()
    at = [i for i, line in enumerate(ir) if re.search(r"call void @llvm\.amdgcn\.wave\.barrier", line)]
    assert at
    for i in at:
        assert 'fence syncscope("wavefront") release' in ir[i - 1], (i, ir[i - 1])
        assert 'fence syncscope("wavefront") acquire' in ir[i + 1], (i, ir[i + 1])
