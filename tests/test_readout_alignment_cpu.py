"""The read-out kernels' wide loads ask for no more alignment than an
amplitude has: a server takes any buffer of amplitudes.  Read off the code the
compiler makes for the device (no GPU is needed)."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2010_09746_amd import build as B


@pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="needs hipcc")
def test_wide_loads_of_a_state_are_aligned_like_its_amplitudes(tmp_path):
    out = tmp_path / "readout.ll"
    subprocess.run([B.HIPCC] + B.HIP_FLAGS + ["--cuda-device-only", "-S", "-emit-llvm", "-x", "hip",
                                              os.path.join(B.CSRC, "readout.hip"), "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    code = out.read_text()
    for kernel, amplitude in (("k_zsumIfE", 8), ("k_zsumIdE", 16)):
        body = re.search(r"^define [^\n]*%s.*?^}" % kernel, code, re.S | re.M).group(0)
        align = [int(a) for a in re.findall(r"load <\d+ x \w+>, ptr addrspace\(1\)[^\n]*?align (\d+)", body)]
        assert align and max(align) <= amplitude
