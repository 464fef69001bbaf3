"""The kernels' prologues divide by numbers of the launch through a multiplier and a shift (csrc/sdpa_fwd_launch.h): exact for every
numerator below 2^31, checked at the edges of the quotients of divisors of every size."""
import shutil
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2603_01960_amd" / "csrc"

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "sdpa_fwd_launch.h"
using namespace tsdpa;
static bool exact(uint32_t d, uint64_t n)
{
    if (n >= 1ull << 31) return true;
    const Divisor by = divisor(d);
    const uint32_t q = (uint32_t)(((uint64_t)(2u * (uint32_t)n) * by.mul) >> 32) >> by.shift;    // as the kernels do it
    if (q == n / d) return true;
    std::printf("%llu / %u gives %u\n", (unsigned long long)n, d, q);
    return false;
}
int main()
{
    std::mt19937_64 rng(7);
    bool ok = true;
    auto check = [&](uint32_t d) {
        const uint64_t last = ((1ull << 31) - 1) / d * d;
        for (uint64_t m : {(uint64_t)0, (uint64_t)d, 2 * (uint64_t)d, last / 2 / d * d, last - d, last})
            for (int64_t e : {-1, 0, 1}) if ((int64_t)m + e >= 0) ok = exact(d, m + e) && ok;
        ok = exact(d, (1ull << 31) - 1) && ok;
        for (int i = 0; i < 8; ++i) ok = exact(d, rng() >> 33) && ok;
    };
    for (uint32_t d = 1; d < 5000; ++d) check(d);
    for (int b = 2; b < 31; ++b) for (int e : {-1, 0, 1}) check((1u << b) + e);
    for (int i = 0; i < 20000; ++i) check(1 + (uint32_t)(rng() % 0x7fffffffull) / (1u << (rng() % 24)));
    return ok ? 0 : 1;
}
"""


def test_quotients_are_exact(tmp_path):
    rocm = Path("/opt/rocm")
    if shutil.which("g++") is None or not (rocm / "include/hip/hip_runtime.h").exists():
        pytest.skip("needs g++ and the HIP headers")
    src, exe = tmp_path / "divisor.cpp", tmp_path / "divisor"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", f"-I{rocm}/include", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert done.returncode == 0, done.stdout[:2000]
