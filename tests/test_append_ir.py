"""An fp8 cache may start at any byte (a view into a larger buffer): the append's
wide accesses of its tiles must not promise the compiler more. Host-only: the
kernels' device code in LLVM's intermediate form, from the library's source and
flags."""

import os
import re
import subprocess

import pytest

from paper_2605_20863_amd import build as B


@pytest.fixture(scope="module")
def append_ir(tmp_path_factory):
    try:
        hipcc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("ir") / "pda_append.ll"
    cmd = [hipcc, f"--offload-arch={B.ARCH}", "-O3", "-std=c++17", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
           *B.HIP_FLAGS, "--cuda-device-only", "-S", "-emit-llvm", os.path.join(B.CSRC, "pda_append.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return out.read_text()


def test_fp8_tile_accesses_promise_no_alignment(append_ir):
    kernels = re.findall(r"^define [^\n]*append_kernel\w*KvTypeE2[^\n]*\{\n(.*?)^\}", append_ir, re.S | re.M)
    assert len(kernels) == 2  # head dims 64 and 128
    for body in kernels:
        wide = re.findall(r"^.*\b(?:load|store) <4 x i32>.*$", body, re.M)
        words = re.findall(r"^.*\bstore i32 .*$", body, re.M)  # (float scales are stored as float)
        assert wide and words
        for line in wide + words:
            assert re.search(r"align 1\b(?!\d)", line), line
