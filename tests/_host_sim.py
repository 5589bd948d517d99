"""The library's host code (pda_host.cpp) built by the host C++ compiler over
the note-taking HIP runtime of tests/hostsim/fake_hip.cpp, called through its C
interface: what a call would launch, in a capture, and when memory is short."""

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2605_20863_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_20863_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
STREAM = 0x1000


def build(out):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the ROCm headers")
    cmd = [gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(CSRC, "pda_host.cpp"), os.path.join(ROOT, "tests", "hostsim", "fake_hip.cpp"), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-4000:]
    return Sim(out)


class Sim:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        self.lib.sim_room.restype = ctypes.c_int64
        self.lib.sim_room.argtypes = [ctypes.c_int64]
        self.lib.sim_allocated.restype = ctypes.c_int64
        self.lib.sim_reset.argtypes = [ctypes.c_ulonglong, ctypes.c_int64]
        self.lib.pda_last_error.restype = ctypes.c_char_p

    def room(self, p):
        return self.lib.sim_room(p)

    def allocated(self):
        return self.lib.sim_allocated()

    def reset(self, capture=0, limit=-1):
        self.lib.sim_reset(capture, limit)

    def _notes(self, fn, *names):
        out = (ctypes.c_int64 * len(names))()
        fn(out)
        return dict(zip(names, out))

    def decode(self, B, hq, hkv, d, kv, blocks, q_tokens=1, max_seq_len=0, options=None, noalloc=False, stream=STREAM):
        """(status, notes on the decode launch)"""
        qt = _lib.F32 if kv == _lib.F32 else _lib.BF16
        pr = _lib.Problem(B, hq, hkv, d, 16, blocks, B * blocks + 1, max_seq_len, qt, kv, qt, q_tokens)
        fn = self.lib.pda_paged_decode_attention_noalloc if noalloc else self.lib.pda_paged_decode_attention
        p = ctypes.c_void_p(0x10000)  # never read
        rc = fn(p, p, p, p, p, p, p, ctypes.c_float(0.1), ctypes.byref(pr),
                None if options is None else ctypes.byref(options), ctypes.c_void_p(stream))
        return rc, self._notes(self.lib.sim_decode, "parts", "clear", "epoch", "hdr")

    def prefill(self, B, T, hq, hkv, d, kv, blocks, num_blocks=None, stream=STREAM):
        """(status, notes on the prefill launch)"""
        pr = _lib.PrefillProblem(B, T, hq, hkv, d, 16, blocks, num_blocks or B * blocks + 1, 0, _lib.BF16, kv, _lib.BF16)
        p = ctypes.c_void_p(0x10000)
        rc = self.lib.pda_paged_prefill_attention(p, p, p, p, p, p, p, p, ctypes.c_float(0.1), ctypes.byref(pr),
                                                  ctypes.c_void_p(stream))
        return rc, self._notes(self.lib.sim_prefill, "slots", "v_img", "k_img", "img_tiles", "list_max", "hdr", "items",
                               "parts", "splits", "part_ml", "part_acc")

    def release(self):
        self.lib.pda_release_workspaces()
