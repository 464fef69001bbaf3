"""Which kernels a backward call takes (csrc/sdpa_bwd_pick.h), evaluated on the host."""
import ctypes
import shutil
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_01960_amd" / "csrc"

EXPORTS = r"""
#include "sdpa_bwd_pick.h"
using namespace tsdpa;
extern "C" {
int joint(int D, int causal, int heads, int group, int S) { return pick_bwd_joint(D, causal != 0, heads, group, S); }
}
"""


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    at = tmp_path_factory.mktemp("pick")
    (at / "pick.cpp").write_text(EXPORTS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", str(at / "pick.cpp"), "-o",
                    str(at / "pick.so")], check=True)
    return ctypes.CDLL(str(at / "pick.so"))


def test_large_grouped_calls_keep_the_passes_apart(pick):
    """Where the launch for the statistics of the query rows costs more than one grid gains."""
    for hkv, G, S in ((96, 4, 4096), (40, 4, 8192), (16, 8, 16384)):
        for D in (64, 96):
            assert pick.joint(D, 0, hkv * G, G, S) == 0 and pick.joint(D, 1, hkv * G, G, S) == 0
    for D, causal, hkv, G, S in ((64, 0, 99, 2, 512), (64, 0, 117, 2, 1241), (64, 0, 44, 2, 2048), (96, 0, 30, 2, 2048),
                                 (64, 1, 77, 4, 3879), (96, 1, 108, 2, 256)):
        assert pick.joint(D, causal, hkv * G, G, S) == 0
