"""Calls of the cache entry points around the lines where their route changes: a decoding step in one run or several (by a
head's K and by the heads), combined by its own workgroups or by the merge kernel (runs just below, at and past the eight that
are loaded at once), and 17 to 32 query rows in streams of K/V tiles or in the decoding kernel, against the float64 oracle with
the usual forward tolerances."""
import pytest

import test_sdpa_kv_gpu as kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,D,Skv", [(1, 64, 1640), (1, 64, 1641), (3, 160, 656), (3, 160, 657), (65, 96, 2083), (65, 96, 2084),
                                         (85, 128, 1600), (86, 128, 1600), (127, 64, 3200), (128, 64, 3200)])
def test_one_run_or_several(heads, D, Skv):
    for Sq, dtype in ((1, "bf16"), (8, "f16")):
        q, k, v = kv.make_q_kv(1, heads, Sq, Skv, D, dtype, seed=7000 + Skv)
        kv.check_kv(q, k, v, dtype, causal=True, tag="default runs")


@pytest.mark.parametrize("D,Sq", [(64, 1), (160, 1), (96, 2), (128, 4), (96, 5), (160, 6), (160, 8), (128, 9), (64, 16)])
def test_runs_combined(D, Sq):
    """Few rows and runs are combined by a head's last workgroup, the others by the merge kernel."""
    q, k, v = kv.make_q_kv(1, 3, Sq, 2300, D, "bf16", seed=7100 + D)
    for splits in (2, 7, 8, 9, 15, 16, 17, 33):
        kv.check_kv(q, k, v, "bf16", splits=splits, tag="runs")
    kv.check_kv_lens(4, 6, 3, Sq, 2300, D, "bf16", [0, 40, 700, 2299], False, 9)     # runs without keys


@pytest.mark.parametrize("heads,rows,Skv,D", [(2, 17, 33, 160), (64, 32, 64, 96), (65, 32, 64, 96), (16, 32, 300, 160), (5, 24, 1023, 160),
                                              (64, 20, 1030, 160), (128, 17, 515, 128), (129, 32, 200, 64), (512, 17, 90, 64), (513, 17, 90, 64),
                                              (256, 18, 70, 128), (257, 18, 70, 128), (66, 20, 4096, 64), (66, 20, 4097, 64), (70, 32, 1300, 160)])
def test_seventeen_to_thirty_two_rows(heads, rows, Skv, D):
    q, k, v = kv.make_q_kv(1, heads, rows, Skv, D, "f16", seed=7200 + heads)
    kv.check_kv(q, k, v, "f16", causal=True, tag="few rows")
    kv.check_kv_lens(2, heads, heads // 2 if heads % 2 == 0 else heads, rows // 2, Skv, D, "bf16", [Skv // 3, Skv], False, 0)


# 128-row query tiles around two per CU: (heads, rows, Skv, D), one or more splits of the key range
@pytest.mark.parametrize("heads,rows,Skv,D", [(27, 1100, 1100, 64), (30, 1100, 1060, 96), (38, 1100, 2050, 64), (2, 200, 100, 128),
                                              (65, 128, 511, 128), (3, 300, 33, 128), (85, 129, 2100, 64), (86, 257, 2100, 64), (171, 129, 2100, 64)])
def test_chunks_around_two_tiles_per_cu(heads, rows, Skv, D):
    q, k, v = kv.make_q_kv(1, heads, rows, Skv, D, "bf16", seed=7300 + rows)
    kv.check_kv(q, k, v, "bf16", causal=Skv >= rows, tag="chunk")


# no mask: 128 rows per workgroup where 256 begin a second round with the last rows half empty, 256 where either is one round
@pytest.mark.parametrize("heads,rows,Skv,D", [(52, 1100, 70, 160), (37, 1600, 33, 160), (16, 3900, 65, 160), (29, 2100, 64, 128), (16, 3901, 40, 128),
                                              (13, 4900, 50, 96), (8, 8000, 45, 96), (30, 2300, 70, 128)])
def test_long_query_blocks_without_a_mask(heads, rows, Skv, D):
    q, k, v = kv.make_q_kv(1, heads, rows, Skv, D, "bf16", seed=7350 + rows)
    kv.check_kv(q, k, v, "bf16", splits=1, tag="long block")


def test_long_caches_in_few_tiles():
    """Splits of one CU's two workgroups each, runs of 512 keys and more."""
    from paper_2603_01960_amd import binding
    for D, Skv in ((64, 8200), (160, 8321)):
        q, k, v = kv.make_q_kv(1, 3, 400, Skv, D, "bf16", seed=7400 + D)
        n = binding.kv_default_splits(1, 3, 400, Skv, D, binding.BF16)
        assert n > 1 and n * 12 <= 2048 and Skv // n >= 512
        kv.check_kv(q, k, v, "bf16", causal=True, tag="long cache")


@pytest.mark.parametrize("heads,rows,Skv,D,given", [(20, 24, 1500, 160, 1), (64, 32, 1024, 160, 1), (202, 128, 1432, 160, 1), (103, 200, 1346, 160, 1),
                                                    (13, 300, 9000, 96, 7), (26, 128, 12000, 160, 10)])
def test_a_workspace_for_fewer_states_is_taken(heads, rows, Skv, D, given):
    """splits = 0 with a workspace (or none) that holds `given` states per tile, fewer than the default count's."""
    import torch
    from paper_2603_01960_amd import binding
    assert binding.kv_default_splits(1, heads, rows, Skv, D, binding.BF16) > given
    size = binding.kv_workspace_bytes(1, heads, rows, D, given)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda") if size else None
    g = torch.Generator("cuda").manual_seed(7450)
    q, k, v = (torch.randn((1, heads, s, D), device="cuda", generator=g).bfloat16() for s in (rows, Skv, Skv))
    o = torch.full_like(q, float("nan"))
    st = binding.load_library().tiled_sdpa_fwd_kv(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), None, 1, heads, rows, Skv, D, float("nan"),
                                                  binding.BF16, torch.cuda.current_stream().cuda_stream, 0, 0, 0, 0,
                                                  ws.data_ptr() if size else None, size)
    assert st == 0, binding.status_string(st)
    torch.testing.assert_close(o.float(), binding.sdpa_kv(q, k, v).float(), rtol=2e-2, atol=2e-2)
    if size:
        assert torch.equal(binding.sdpa_kv(q, k, v, workspace=ws), o)
    st = binding.load_library().tiled_sdpa_fwd_kv(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), None, 1, heads, rows, Skv, D, float("nan"),
                                                  binding.BF16, torch.cuda.current_stream().cuda_stream, 0, 0, 0, given + 1, ws.data_ptr() if size else None, size)
    assert st != 0                                # a count of the caller's own is not lowered


def test_without_a_workspace_the_count_is_one_that_fits():
    """26 heads of 128 rows at D = 160: the default count's states exceed the library's own buffer, a smaller count's do not."""
    import torch
    from paper_2603_01960_amd import binding
    H, Sq, Skv, D = 26, 128, 12000, 160
    n = binding.kv_default_splits(1, H, Sq, Skv, D, binding.BF16)
    assert binding.kv_workspace_bytes(1, H, Sq, D, n) > binding.STATIC_SCRATCH_BYTES
    g = torch.Generator("cuda").manual_seed(7500)
    q, k, v = (torch.randn((1, H, s, D), device="cuda", generator=g).bfloat16() for s in (Sq, Skv, Skv))
    o = torch.full_like(q, float("nan"))
    st = binding.tiled_sdpa_fwd_kvcache_static(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), None, None, 1, H, H, Sq, Skv, D,
                                               float("nan"), binding.BF16, torch.cuda.current_stream().cuda_stream, 0, 0, 0, 0)
    assert st == 0, binding.status_string(st)
    assert torch.equal(o, binding.sdpa_kv(q, k, v, splits=10))       # one workgroup per CU: 256 / 26, rounded up


# One run where the decoding kernel had several, and streams of more than 64 heads, multiply each weight as two 16-bit halves (the
# largest weight of a wavefront is exact anyway, and wavefronts with a tile or two each had many of those).  The least error is the
# rounding of the result, measured on the exact one; rounded weights add as much again (in the squares), weights rounded in
# halves a quarter of that: sqrt(1.25).  At D = 160 the decoding kernel keeps its runs of a tile per wavefront past 256 keys:
# weights rounded but for the largest of 32 normal scores, 27 % of the sum of squares, so sqrt(1 + 0.73).  3 % for the
# spread of a few hundred values.
HALVES = 1.118


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("heads,rows,Skv,D,rounded", [
    (16, 2, 744, 96, HALVES), (2, 8, 1473, 64, HALVES), (7, 16, 760, 128, HALVES), (9, 1, 635, 160, HALVES), (36, 5, 257, 128, HALVES),
    (70, 2, 2040, 96, HALVES),
    (20, 3, 260, 160, HALVES), (72, 20, 512, 128, HALVES), (112, 32, 385, 96, HALVES), (72, 24, 900, 64, HALVES), (65, 17, 257, 64, HALVES),
    (66, 20, 3000, 128, HALVES), (3, 24, 717, 160, 1.315), (16, 23, 807, 160, 1.315)])
def test_error_of_few_rows(heads, rows, Skv, D, rounded, paged):
    import torch
    from paper_2603_01960_amd import binding
    for dtype in (torch.bfloat16, torch.float16):
        g = torch.Generator("cuda").manual_seed(7600 + heads)
        q, k, v = (torch.randn((1, heads, n, D), device="cuda", generator=g).to(dtype) for n in (rows, Skv, Skv))
        if paged:
            block, pages = 64, -(-Skv // 64)
            pool = torch.full((2, pages, heads, block, D), float("nan"), device="cuda", dtype=dtype)
            for side, x in zip(pool, (k, v)):
                for i in range(pages):
                    part = x[0, :, i * block:(i + 1) * block]
                    side[pages - 1 - i, :, :part.shape[1]] = part
            table = torch.arange(pages - 1, -1, -1, device="cuda", dtype=torch.int32)[None].contiguous()
            o = binding.sdpa_paged(q, pool[0], pool[1], torch.tensor([Skv], device="cuda", dtype=torch.int32), table)
        else:
            o = binding.sdpa_kv(q, k, v)
        err = least = 0.0
        for h in range(heads):
            want = (q[0, h].double() @ k[0, h].double().t().contiguous() * D ** -0.5).softmax(-1) @ v[0, h].double()
            err += ((o[0, h].double() - want) ** 2).sum().item()
            least += ((want.to(dtype).double() - want) ** 2).sum().item()
        assert err ** 0.5 <= 1.03 * rounded * least ** 0.5, f"{dtype} {(err / least) ** 0.5:.3f} times the rounding of the result"


def test_an_infinite_value_stays_one():
    import torch
    from paper_2603_01960_amd import binding
    for heads, rows, Skv, D in ((3, 4, 600, 96), (70, 20, 600, 64)):
        for dtype in (torch.bfloat16, torch.float16):
            g = torch.Generator("cuda").manual_seed(7700)
            q, k, v = (torch.randn((1, heads, n, D), device="cuda", generator=g).to(dtype) for n in (rows, Skv, Skv))
            v[0, :, 300, 5] = float("inf")
            o = binding.sdpa_kv(q, k, v)
            assert (o[..., 5] == float("inf")).all()
            assert torch.isfinite(o[..., :5]).all() and torch.isfinite(o[..., 6:]).all()
