"""In-kernel hand-overs between workgroups (a flag or a count that others poll):
the flag follows a release fence of one thread, which drains that thread's
wavefront only, so every wavefront has to drain its own stores before the
barrier in front of it.  Read off the device code of the built library."""
from __future__ import annotations

import glob
import os
import re
import shutil
import subprocess

import pytest

import paper_0903_5067_amd as lbm

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _device_code(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(lbm.LIB_PATH):
        pytest.skip("liblbmd.so not built")
    so = shutil.copy(lbm.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", so], cwd=tmp_path, check=True, capture_output=True)
    kernel, out = None, {}
    for f in glob.glob(str(tmp_path / "*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                kernel = out.setdefault(m[1], [])
            elif kernel is not None and line.startswith("\t"):
                kernel.append(line.split("//")[0].strip())
    return out


def test_every_wavefront_drains_its_stores_before_a_release(tmp_path):
    releases = 0
    for name, code in _device_code(tmp_path).items():
        for i, ins in enumerate(code):
            if not ins.startswith("buffer_wbl2"):   # a release beyond the workgroup
                continue
            releases += 1
            bar = max(k for k in range(i) if code[k] == "s_barrier")
            assert any(re.fullmatch(r"s_waitcnt .*vmcnt\(0\).*", c) for c in code[bar - 6:bar]), (name, code[bar - 8:i + 1])
    assert releases >= 14   # k_step: six kernels; k_collide_headed: four, two each
