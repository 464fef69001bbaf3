"""The decoding kernel (at most 32 query rows per key/value head, tile left to the library) at the edges of its tiles (32 keys,
16 query rows), of its wavefronts' shares (4 or 8 tiles per round) and of its runs, against the float64 oracle: the
usual forward tolerances."""
import pytest

import test_sdpa_kv_gpu as kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128, 160])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_row_and_key_counts_around_the_tiles(D, dtype):
    for Sq in (1, 15, 16, 17, 32):
        for Skv in (1, 31, 32, 33, 129, 257, 700):
            q, k, v = kv.make_q_kv(1, 2, Sq, Skv, D, dtype, seed=4000 + 100 * Sq + Skv)
            # one run (four or eight wavefronts), runs the kernel combines itself or leaves to the merge, empty runs
            for splits in (1, 3, 40):
                kv.check_kv(q, k, v, dtype, splits=splits, tag="decode")
            if Skv >= Sq:
                kv.check_kv(q, k, v, dtype, splits=2, causal=True, tag="decode causal")


@pytest.mark.parametrize("splits", [0, 1, 2, 5])
@pytest.mark.parametrize("D,G,Sq", [(64, 8, 1), (128, 4, 2), (160, 8, 4), (96, 1, 3)])
def test_grouped_heads_lengths_and_pages(splits, D, G, Sq):
    lens = [0, 1, 130, 513, 1000, 64, 999]
    for causal in (False, True):
        kv.check_kv_lens(len(lens), 2 * G, 2, Sq, 1000, D, "bf16", lens, causal, splits)
        kv.check_paged(len(lens), 2 * G, 2, Sq, D, "bf16", lens, 64, causal, splits)


@pytest.mark.parametrize("entries", [2, 63, 64, 65])
def test_runs_follow_the_longest_entry(entries):
    """Runs are cut by the longest of up to 64 entries, by each entry's own length beyond: the longest one first, last and in the
    middle, lengths around four tiles per run, most of the capacity unused."""
    for splits in (2, 5, 40):
        for at, most in ((0, 1500), (entries - 1, 128 * splits - 63), (entries // 2, 128 * splits + 1)):
            lens = [(11 * i) % 97 for i in range(entries)]
            lens[at] = min(most, 2900)
            kv.check_kv_lens(entries, 4, 2, 1, 3000, 64, "bf16", lens, True, splits)
            kv.check_paged(entries, 2, 2, 3, 128, "f16", lens, 64, False, splits)


def test_more_workgroups_than_fit_at_once():
    # 600 key/value heads (four wavefronts each), 300 heads in two runs
    q, k, v = kv.make_q_kv(100, 6, 1, 300, 64, "bf16", seed=4900)
    kv.check_kv(q, k, v, "bf16", tag="many heads")
    # (17 to 32 rows stay with this kernel from 65 heads on)
    for D in (64, 96, 128, 160):
        q, k, v = kv.make_q_kv(11, 6, 17 + D // 32 * 3, 300, D, "bf16", seed=4902)
        kv.check_kv(q, k, v, "bf16", splits=D // 64, causal=True, tag="many heads of many rows")
    q, k, v = kv.make_q_kv(50, 6, 2, 300, 128, "f16", seed=4901)
    kv.check_kv(q, k, v, "f16", splits=2, causal=True, tag="many heads, two runs")


def test_output_buffer_holds_nothing_but_the_result():
    """The runs' marks stand in the output until the result replaces them: whatever the buffer held before, an earlier result
    of the same call included, must not matter."""
    import torch
    from paper_2603_01960_amd import binding
    q, k, v = (t.cuda() for t in kv.make_q_kv(2, 3, 4, 2000, 128, "bf16", seed=4950))
    ref = binding.sdpa_kv(q, k, v, splits=8)
    for fill in (float("nan"), 0.0, 1.0):
        out = torch.full_like(q, fill)
        for _ in range(3):
            assert torch.equal(binding.sdpa_kv(q, k, v, splits=8, out=out), ref)


def test_nan_rows_stay_nan_however_the_runs_are_combined():
    """A query row with a NaN has NaN weights: its output is NaN and no other row's is, whether one run, the kernel itself
    or either merge kernel (few rows, many rows) makes the result; runs without keys (lens) change nothing."""
    import torch
    from paper_2603_01960_amd import binding
    for B, Sq, splits in ((2, 4, 1), (2, 4, 8), (2, 4, 40), (700, 4, 3)):
        q, k, v = (t.cuda() for t in kv.make_q_kv(B, 1, Sq, 400, 64, "bf16", seed=4970))
        lens = torch.full((B,), 150, dtype=torch.int32, device="cuda")
        for kv_lens in (None, lens):
            ref = binding.sdpa_kv(q, k, v, splits=splits, kv_lens=kv_lens)
            bad = q.clone()
            bad[1, 0, 2, 5] = float("nan")
            out = binding.sdpa_kv(bad, k, v, splits=splits, kv_lens=kv_lens)
            assert out[1, 0, 2].isnan().all(), (B, splits)
            out[1, 0, 2] = ref[1, 0, 2]
            # (the NaN makes its wavefront raise every row's reference: other roundings of the weights, 2^-9 each)
            torch.testing.assert_close(out.float(), ref.float(), rtol=1e-2, atol=1e-2)


def test_arguments_that_leave_a_choice_open():
    """splits=None is the library's choice, as 0; of a longer `grads` the first three are used."""
    import torch
    from paper_2603_01960_amd import binding
    q, k, v = (t.cuda() for t in kv.make_q_kv(1, 2, 64, 64, 64, "f16", seed=4980))
    ref = binding.sdpa_kv(q, k, v)
    assert torch.equal(binding.sdpa_kv(q, k, v, splits=None), ref)
    o, lse = binding.sdpa(q, k, v, return_lse=True)
    want = binding.sdpa_backward(q, k, v, o, q, lse)
    grads = [torch.empty_like(t) for t in (q, k, v)] + [None]
    assert binding.sdpa_backward(q, k, v, o, q, lse, grads=grads) is grads
    assert all(torch.equal(a, b) for a, b in zip(grads, want))
