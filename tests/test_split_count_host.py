"""The split count that the library picks never falls as a cache grows: a workspace sized once, for the capacity, then holds the
states of every length on the way there (a call whose count does not fit its workspace is refused)."""
import ctypes

import pytest

from paper_2603_01960_amd import binding

LENGTHS = sorted({*range(32, 2100, 97), *range(2048, 33000, 448), 511, 512, 1023, 1024, 2047, 2049, 4096, 4097, 8192, 8193, 15872, 16384,
                  32000, 32768})
HEADS = [1, 2, 5, 8, 13, 16, 24, 31, 33, 48, 63, 64, 65, 72, 85, 96, 127, 128, 152, 200, 255, 256, 272, 300, 341, 342, 511, 512]


def _of_tile(heads, rows, n, D):
    splits = ctypes.c_int(0)
    assert binding.load_library().tiled_sdpa_kv_tile_splits(1, heads, rows, n, D, binding.BF16, 0, 128, 64, ctypes.byref(splits)) == 0
    return splits.value


def _default(heads, rows, n, D):
    return binding.kv_default_splits(1, heads, rows, n, D, binding.BF16)


@pytest.mark.parametrize("D", [64, 96, 128, 160])
@pytest.mark.parametrize("rows", [1, 8, 17, 32, 65, 128, 129, 300, 1024])
def test_a_longer_cache_has_no_fewer_splits(D, rows):
    for heads in HEADS:
        for count in (_default, _of_tile):
            most = at = 0
            for n in LENGTHS:
                splits = count(heads, rows, n, D)
                assert splits >= most, f"{heads} heads of {rows} rows: {most} splits of {at} keys, {splits} of {n}"
                most, at = splits, n


def test_workspace_of_the_default_count_is_bounded():
    """At most four rounds of 512 workgroups, 128 rows of states each."""
    for D in (64, 160):
        for rows in (1, 32, 64, 128, 129, 512, 4096):
            for heads in HEADS:
                for n in (2048, 16384, 131072):
                    states = binding.kv_default_splits(1, heads, rows, n, D, binding.BF16)
                    size = binding.kv_workspace_bytes(1, heads, rows, D, states)
                    assert size <= 2048 * 128 * (D + 2) * 4
