"""What the compiler cannot know of instructions written in assembly, checked on its own output (no GPU): which registers they write, and the
wait states that the hardware wants between two instructions, which the compiler inserts for its own instructions only.  Small kernels that put the
wrappers where their neighbours are closest, and the kernels that use them."""
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2603_01960_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not Path(HIPCC).exists(), reason="hipcc not available")

# translation units with kernels that use them
UNITS = [CSRC / f"sdpa_bwd_{x}.hip" for t in ("f16", "bf16") for x in (f"chain_{t}_d64", f"chain_{t}_d96", f"chain_{t}_d128", f"{t}_d64")]

PRELUDE = '#include "sdpa_bwd_chain_kernel.h"\nusing namespace tsdpa;\n'


def assembly(src: Path, out: Path):
    """The instructions of a translation unit, [(name, operands, written in assembly)], labels as names with a colon."""
    from paper_2603_01960_amd import build as lib_build
    done = subprocess.run([HIPCC, *lib_build.FLAGS, *lib_build.extra_flags(src), "-S", "--cuda-device-only", str(src), "-o", str(out)],
                          capture_output=True, text=True, timeout=600)
    assert done.returncode == 0, done.stderr
    code, by_hand = [], False
    for line in out.read_text().split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            by_hand = "#ASMSTART" in line
            continue
        line = line.split(";")[0].strip()
        if not line or (line.startswith(".") and not line.endswith(":")):
            continue
        name, _, rest = line.partition(" ")
        operands = [x.strip() for x in rest.split(",")] if rest else []
        if operands:
            operands[-1:] = operands[-1].split()          # (modifiers)
        code.append((name, operands, by_hand))
    return code


def probe(tmp_path, body):
    """Assembly of a kernel, built with the flags of the five-product backward."""
    src = tmp_path / "sdpa_bwd_chain_probe.hip"
    src.write_text(PRELUDE + body)
    return assembly(src, tmp_path / "probe.s")


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    at = tmp_path_factory.mktemp("units")
    with ThreadPoolExecutor(len(UNITS)) as pool:
        return dict(zip((u.name for u in UNITS), pool.map(lambda u: assembly(u, at / (u.stem + ".s")), UNITS)))


def registers(operand):
    """{("s", 4), ("s", 5)} of s[4:5]"""
    m = re.match(r"([vas])(?:(\d+)|\[(\d+):(\d+)\])$", operand)
    if not m:
        return set()
    first, last = (m[2], m[2]) if m[2] else (m[3], m[4])
    return {(m[1], i) for i in range(int(first), int(last) + 1)}


def before(code, at, states):
    """The instructions up to `states` wait states before instruction `at`, nearest first.  (Straight back in the listing: what stands between
    an instruction in assembly and its neighbours does so on every way to it.)"""
    i = at - 1
    while i >= 0 and states > 0:
        name, operands, _ = code[i]
        if not name.endswith(":"):
            yield code[i]
            states -= int(operands[0]) + 1 if name == "s_nop" else 1
        i -= 1


def late_scalars(code):
    """Memory instructions in assembly less than five wait states after a vector instruction that writes a scalar register they read."""
    found, seen = [], 0
    for i, (name, operands, by_hand) in enumerate(code):
        if by_hand and name.startswith("buffer_"):
            seen += 1
            used = {r for x in operands for r in registers(x) if r[0] == "s"}
            found += [(code[i], other) for other in before(code, i, 5) if other[0].startswith("v_") and registers(other[1][0]) & used]
    return found, seen


def late_operands(code):
    """Matrix instructions in assembly less than two wait states after a vector instruction that writes a register they read."""
    found, seen = [], 0
    for i, (name, operands, by_hand) in enumerate(code):
        if by_hand and name.startswith("v_mfma"):
            seen += 1
            used = set().union(*(registers(x) for x in operands[1:]))
            found += [(code[i], other) for other in before(code, i, 2)
                      if other[0].startswith("v_") and not other[0].startswith("v_mfma") and registers(other[1][0]) & used]
    return found, seen


def early_results(code):
    """Instructions of the compiler's that touch an accumulator less than 19 wait states after a matrix instruction in assembly that writes it."""
    found, seen = [], 0
    for i, (_, operands, by_hand) in enumerate(code):
        touched = {r for x in operands for r in registers(x) if r[0] == "a"}
        if not by_hand and touched:
            seen += 1
            found += [(code[i], other) for other in before(code, i, 19)
                      if other[2] and other[0].startswith("v_mfma") and registers(other[1][0]) & touched]
    return found, seen


def test_m0_of_the_compilers_loads_survives_a_load_in_assembly(tmp_path):
    """A load to the LDS takes its address from m0, which the compiler sets once for loads to the same place: not past a load in assembly."""
    code = probe(tmp_path, r"""
__global__ void loads(int *p, int bytes, int at, int other)
{
    extern __shared__ unsigned char smem[];
    const lds_ptr lds = (lds_ptr)smem;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, bytes, 0x00020000);
    const int voff = threadIdx.x * 4;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(lds + at), 4, voff, 0, 0, 0);
    lds_load16(rsrc, other, voff, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(lds + at), 4, voff, 64, 0, 0);
    lds_load4(rsrc, other, voff, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(lds + at), 4, voff, 128, 0, 0);
    lds_load4_agent(rsrc, other);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (TSDPA_LDS void *)(lds + at), 4, voff, 192, 0, 0);
}
""")
    loads = set_by = 0
    for name, operands, by_hand in code:
        if operands and operands[0] == "m0":
            set_by = by_hand
        if name.startswith("buffer_load") and "lds" in operands:
            loads += 1
            assert set_by == by_hand, f"load {loads} has the m0 of the one before it"
    assert loads == 7


def test_loads_in_assembly_wait_for_scalar_registers_that_vector_instructions_write(tmp_path, units):
    code = probe(tmp_path, r"""
__global__ void loads(const int *words, int lane, int dst)
{
    const int x = words[threadIdx.x];
    auto word = [&](int i) __attribute__((always_inline)) { return __builtin_amdgcn_readlane(x, lane + i); };
    auto rsrc = [&](int i) __attribute__((always_inline)) {
        void *at = (void *)((unsigned long long)(unsigned)word(i) | (unsigned long long)(unsigned)word(i + 1) << 32);
        return __builtin_amdgcn_make_buffer_rsrc(at, (short)0, word(i + 2), 0x00020000);
    };
    lds_load16(rsrc(0), dst, 0, word(3));
    lds_load4(rsrc(4), dst, 0, word(7));
    lds_load4_agent(rsrc(8), dst);
}
""")
    found, seen = late_scalars(code)
    assert seen == 3 and not found, found
    for name, code in units.items():
        found, seen = late_scalars(code)
        assert seen > 0 and not found, f"{name}: {found}"


@pytest.mark.parametrize("vec,elem", [("f16x8", "_Float16"), ("bf16x8", "__bf16")])
def test_matrix_instructions_in_assembly_keep_their_distances(tmp_path, vec, elem):
    code = probe(tmp_path, r"""
__global__ void products(const u32x4 *in, float *out, unsigned x)
{
    f32x16 k[2][1], v[2][1];
#pragma unroll
    for (int i = 0; i < 16; ++i) k[0][0][i] = k[1][0][i] = v[0][0][i] = v[1][0][i] = 0.f;
    const u32x4 a = in[threadIdx.x], b = in[threadIdx.x + 64];
    auto made = [&](const u32x4 &y) __attribute__((always_inline)) { return __builtin_bit_cast(VEC, y); };
    for (unsigned i = 0; i < 3; ++i) AccMfma<ELEM>::run(k[0][0], k[1][0], made(a ^ (x + i)), made(b ^ (x - i)), made(b + (x ^ i)));
    AccMfma<ELEM>::run(v[0][0], v[1][0], made(a), made(a), made(b));
    settle(k, v);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += k[0][0][i] * k[1][0][i] + v[0][0][i] * v[1][0][i];
    out[threadIdx.x] = sum;
}
""".replace("VEC", vec).replace("ELEM", elem))
    for check in (late_operands, early_results):
        found, seen = check(code)
        assert seen >= 2 and not found, f"{check.__name__}: {found}"


@pytest.mark.parametrize("check", [late_operands, early_results])
def test_matrix_instructions_of_the_kernels_keep_their_distances(units, check):
    for name, code in units.items():
        if "chain" in name:
            found, seen = check(code)
            assert seen > 0 and not found, f"{name}: {found}"
