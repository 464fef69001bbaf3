"""No C++ exception may leave a C entry point: the decoding call's ticket is drawn without the system's random source where that
fails.  Host only (no GPU is visible to the child, whose call ends at the launch)."""
import os
import subprocess
import sys
from pathlib import Path

import pytest

from paper_2603_01960_amd import binding

SOURCE = r"""
#include <random>
#include <stdexcept>
// stands in for the C++ library's: a system without any random source
namespace std {
void random_device::_M_init(const string &) { throw runtime_error("no random source"); }
random_device::result_type random_device::_M_getval() { throw runtime_error("no random source"); }
void random_device::_M_fini() {}
}
"""

CHILD = """
import ctypes, math, os, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, ci = ctypes.c_void_p, ctypes.c_int
lib.tiled_sdpa_fwd_kv.argtypes = [vp] * 5 + [ci] * 5 + [ctypes.c_float, ci, vp, ci, ci, ctypes.c_uint, ci, vp, ctypes.c_ulonglong]
P = 0x1000
for _ in range(2):
    print("status", lib.tiled_sdpa_fwd_kv(P, P, P, P, None, 1, 1, 1, 4096, 64, math.nan, 1, None, 0, 0, 0, 4, P, 1 << 20), flush=True)
"""


def test_a_missing_random_source_does_not_end_the_process(tmp_path):
    import torch
    if torch.cuda.is_available():
        pytest.skip("the child's pointers are not real: host only")
    src, shim = tmp_path / "norandom.cpp", tmp_path / "norandom.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-shared", "-fPIC", "-w", str(src), "-o", str(shim)], check=True)
    done = subprocess.run([sys.executable, "-c", CHILD, str(shim), str(binding.library_path())], capture_output=True, text=True, timeout=120,
                          env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert done.returncode == 0, done.stderr[-1000:]
    assert done.stdout.split("\n")[:2] == ["status 8", "status 8"]          # the launch, where no GPU is
