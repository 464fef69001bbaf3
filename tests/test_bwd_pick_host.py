"""Which kernels a backward call takes (csrc/sdpa_bwd_pick.h), evaluated on the host: the large calls that keep the passes apart, and
that the cases of the GPU tests between them meet every kernel that some call takes."""
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
int one_launch(int D, int heads, int S) { return bwd_in_one_launch(D, heads, S); }
int chain(int D, int causal, int heads, int group, int S) { return pick_bwd_chain(D, causal != 0, heads, group, S); }
int pairs(int causal, int heads, int group, int S) { return pick_bwd_pairs(causal != 0, heads, group, S); }
// wavefronts along the rows and streams of a pass in a launch of its own, as two digits
int apart(int D, int causal, int keys, int heads, int group, int S)
{
    const long long own = keys ? heads / group : heads;
    if (D == 96 || D == 128) {
        const BwdForm f = pick_bwd_form(D, causal != 0, keys != 0, own * ((S + 127) / 128), (keys ? group : 1) * ((S + 31LL) / 32));
        if (f.ns > 1) return f.nw * 10 + f.ns;
    }
    return D == 128 && !causal && bwd_wide_rows(own, S) ? 81 : 41;
}
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


def kernels(pick, D, causal, hkv, G, S, sums=True):
    """The kernels of a call, as tiled_sdpa_bwd_gqa (csrc/tiled_sdpa.hip) and launch_bwd (csrc/sdpa_bwd_inst.h) take them, with a workspace for the
    sums of dQ or without; the forms with streams of keys, and the passes with streams, are one kernel for grouped and other heads."""
    heads = hkv * G
    if sums and pick.chain(D, causal, heads, G, S):
        return {("five products", D)}
    if D <= 96 and G == 1 and S <= 256 and pick.one_launch(D, heads, S):
        if D == 64 and S > 128 and heads > 256:
            return {("heads one after another", causal)}
        return {("one launch", D, 2 if S <= 64 else 4 if S <= 128 else 8, causal)}
    form = pick.joint(D, causal, heads, G, S)
    if form:
        return {("joint", D, form, "any heads" if form % 10 > 1 else "grouped" if G > 1 else "ungrouped")}
    heads_of = lambda f: "any heads" if f % 10 > 1 else "grouped" if G > 1 else "ungrouped"
    dq = pick.apart(D, causal, 0, heads, G, S)
    dkv = pick.pairs(causal, heads, G, S) if D == 160 else pick.apart(D, causal, 1, heads, G, S)
    return {("dQ", D, dq, heads_of(dq)), ("dK + dV", D, dkv, heads_of(dkv))}


def test_large_grouped_calls_keep_the_passes_apart(pick):
    """Where the launch for the statistics of the query rows costs more than one grid gains."""
    for hkv, G, S in ((96, 4, 4096), (40, 4, 8192), (16, 8, 16384)):
        for D in (64, 96):
            assert pick.joint(D, 0, hkv * G, G, S) == 0 and pick.joint(D, 1, hkv * G, G, S) == 0
    for D, causal, hkv, G, S in ((64, 0, 99, 2, 512), (64, 0, 117, 2, 1241), (64, 0, 44, 2, 2048), (96, 0, 30, 2, 2048),
                                 (64, 1, 77, 4, 3879), (96, 1, 108, 2, 256)):
        assert pick.joint(D, causal, hkv * G, G, S) == 0


def test_calls_that_five_products_make_slower_keep_the_passes(pick):
    """Shapes at which they took 1.01 to 1.07 of the passes' time, on average over both types; others near by, at which they take 0.89 to 0.98, keep them."""
    for D, causal, hkv, G, S in ((64, 0, 128, 3, 512), (64, 0, 128, 4, 512), (64, 0, 64, 2, 1024), (64, 0, 142, 4, 2048), (64, 0, 192, 1, 1024), (64, 0, 206, 8, 1408),
                                 (64, 0, 256, 4, 1371), (64, 1, 63, 1, 4664), (64, 1, 128, 1, 4096), (64, 1, 128, 1, 4160), (96, 1, 64, 1, 2432),
                                 (96, 1, 124, 1, 2432), (96, 1, 128, 1, 2048), (96, 1, 222, 1, 2048), (96, 1, 240, 1, 2048)):
        assert pick.chain(D, causal, hkv * G, G, S) == 0, (D, causal, hkv, G, S)
    for D, causal, hkv, G, S in ((64, 0, 128, 2, 1024), (64, 0, 32, 3, 1936), (64, 0, 128, 1, 2048), (64, 1, 32, 1, 4096), (64, 1, 32, 1, 8192), (96, 1, 128, 1, 3456),
                                 (128, 1, 64, 1, 2048), (128, 0, 64, 1, 1024)):
        assert pick.chain(D, causal, hkv * G, G, S) > 0, (D, causal, hkv, G, S)


def test_the_gpu_cases_meet_every_kernel(pick):
    """In either type: the forms' cases alternate between the types, the others run in both."""
    from test_bwd_chain_gpu import CASES as chain
    from test_bwd_forms_gpu import CASES as forms
    from test_bwd_joint_gpu import CASES as joint

    met = set()
    add = lambda types, kinds: met.update((t, k) for t in types for k in kinds)
    both = ("f16", "bf16")
    for causal in (False, True):
        for D, hkv, G, S in joint:
            add(both, kernels(pick, D, causal, hkv, G, S))
        for D in (64, 96, 128, 160):
            for i, (hkv, G, S) in enumerate(forms):
                add(both[i % 2:i % 2 + 1], kernels(pick, D, causal, hkv, G, S))
        # test_passes_where_the_workspace_has_no_room_for_the_sums
        for D, hkv, G, S in [*joint, *((D, *c) for D in (64, 96, 128) for c in forms)]:
            if pick.chain(D, causal, hkv * G, G, S):
                add(both, kernels(pick, D, causal, hkv, G, S, sums=False))
        # test_one_head_after_another
        for heads, S in ((257, 256), (768, 197)):
            add(both, kernels(pick, 64, causal, heads, 1, S))
    for D, hkv, G, S, causal in chain:
        assert kernels(pick, D, causal, hkv, G, S) == {("five products", D)}
        add(both, kernels(pick, D, causal, hkv, G, S))
    heads = sorted({round(1.15 ** i) for i in range(51)})
    lengths = sorted({round(16 * 1.1 ** i) for i in range(73)} | {1, 32, 33, 64, 65, 128, 129, 256, 257, 512, 1024, 2048, 4096, 8192})
    missed = {}
    for D in (64, 96, 128, 160):
        for causal in (False, True):
            for G in (1, 2, 3, 4, 8, 16):
                for hkv in heads:
                    for S in lengths:
                        for sums in (True, False):
                            for k in kernels(pick, D, causal, hkv, G, S, sums):
                                for t in both:
                                    if (t, k) not in met:
                                        missed.setdefault((t, k), (causal, hkv, G, S, sums))
    assert not missed, f"kernels that no case meets, each with a call that takes it: {missed}"
