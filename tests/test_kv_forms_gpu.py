"""Query blocks against a cache run on streams of K/V tiles where the workgroups are few (up to 192 of 128 rows): every form, dense
and paged, with entries that are empty, shorter than the query block, or end inside the first tiles, and with the split
count left open or given, against the float64 oracle: the usual forward tolerances."""
import pytest

import test_sdpa_kv_gpu as kv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128, 160])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_ragged_caches(D, splits):
    # 32-row workgroups; folded heads whose rows no tile divides; 64-row ones (70 and 150 workgroups of 128 rows)
    for causal in (False, True):
        kv.check_kv_lens(4, 4, 2, 37, 2048, D, "bf16", [0, 20, 700, 2048], causal, splits)
        kv.check_paged(4, 4, 2, 37, D, "bf16", [0, 20, 700, 1990], 64, causal, splits)
    kv.check_kv_lens(35, 2, 2, 40, 1024, D, "f16", [(29 * i) % 1025 for i in range(35)], True, splits)
    kv.check_paged(75, 2, 2, 33, D, "bf16", [(37 * i) % 513 for i in range(75)], 128, True, splits)


@pytest.mark.parametrize("D,dtype", [(64, "f16"), (96, "bf16"), (128, "f16"), (160, "bf16")])
def test_dense_caches(D, dtype):
    for B, H, Sq, Skv in ((1, 1, 33, 65), (1, 2, 100, 129), (1, 3, 64, 4096), (2, 1, 129, 2500), (1, 1, 40, 9000), (1, 66, 50, 700), (1, 70, 40, 1100)):
        q, k, v = kv.make_q_kv(B, H, Sq, Skv, D, dtype, seed=9000 + Sq)
        kv.check_kv(q, k, v, dtype, causal=True, tag="streams causal")
        kv.check_kv(q, k, v, dtype, tag="streams")


@pytest.mark.parametrize("D,dtype", [(64, "bf16"), (96, "f16"), (128, "bf16"), (160, "f16")])
def test_causal_order_of_streams(D, dtype):
    """More than 256 workgroups of 64 rows: the long-tiles-first order beside streams; whole and folded heads, an entry of every
    length."""
    q, k, v = kv.make_q_kv(1, 70, 256, 1100, D, dtype, seed=9100)
    kv.check_kv(q, k, v, dtype, causal=True, tag="streams, ordered")
    kv.check_kv_lens(35, 8, 2, 64, 1024, D, dtype, [(31 * i) % 1025 for i in range(35)], True, 0)
    kv.check_kv_lens(24, 12, 3, 50, 1100, D, dtype, [1100 - 45 * i for i in range(24)], True, 2)


@pytest.mark.parametrize("splits", [2, 3, 4, 5, 8, 9, 17])
def test_merge_of_many_rows(splits):
    """More than 2048 rows: the merge that walks the splits four at a time, with every remainder; under the mask some splits
    have no key of a row."""
    for D, dtype in ((64, "f16"), (160, "bf16")):
        q, k, v = kv.make_q_kv(3, 1, 700, 900, D, dtype, seed=9200 + splits)
        kv.check_kv(q, k, v, dtype, splits=splits, causal=splits % 2 == 0, tag="merge, many rows")
