"""A call against a cache with a tile of the caller's and the split count left open: the count suits the tile (not the decoding kernel
or the streams, which such a call never takes), the tensor functions and the C-ABI agree on it, and a workspace sized by the default
count is enough."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

# (B, H, Hkv, Sq, Skv, D, tile): streams with the tile open; the decoding kernel; grouped heads; no split either way
SHAPES = [(1, 8, 8, 40, 1500, 64, (64, 64)), (1, 160, 160, 1, 8192, 64, (64, 64)), (1, 160, 160, 1, 4000, 128, (64, 32)),
          (2, 16, 4, 20, 3000, 96, (64, 32)), (1, 4, 4, 300, 4096, 160, (128, 32)), (1, 600, 600, 64, 100, 64, (64, 32))]


def _count(binding, B, H, Hkv, Sq, Skv, D, tile):
    n = ctypes.c_int(0)
    assert binding.load_library().tiled_sdpa_kv_tile_splits(B, Hkv, H // Hkv * Sq, Skv, D, binding.BF16, 0, *tile, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("B,H,Hkv,Sq,Skv,D,tile", SHAPES)
def test_both_interfaces_take_the_count_of_the_tile(B, H, Hkv, Sq, Skv, D, tile):
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(Sq + Skv)
    draw = lambda h, s: torch.randn((B, h, s, D), device="cuda", generator=g).bfloat16()
    q, k, v = draw(H, Sq), draw(Hkv, Skv), draw(Hkv, Skv)
    n = _count(binding, B, H, Hkv, Sq, Skv, D, tile)
    default = binding.kv_default_splits(B, Hkv, H // Hkv * Sq, Skv, D, binding.BF16)
    assert _count(binding, B, H, Hkv, Sq, Skv, D, (0, 0)) == default
    want = binding.sdpa_kv(q, k, v, splits=n, tile=tile)
    assert torch.equal(binding.sdpa_kv(q, k, v, tile=tile), want)

    def c_call(nbytes):
        out = torch.full_like(q, float("nan"))
        ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
        st = binding.tiled_sdpa_fwd_gqa(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), None, B, H, Hkv, Sq, Skv, D, float("nan"),
                                        binding.BF16, torch.cuda.current_stream().cuda_stream, *tile, 0, 0, ws.data_ptr() if nbytes else None,
                                        nbytes)
        assert st == 0
        return out
    need = lambda splits: binding.kv_workspace_bytes(B, H, Sq, D, splits)
    assert torch.equal(c_call(need(n)), want)
    # the default count's workspace: that many splits if the tile's own would not fit
    small = c_call(need(default))
    assert torch.equal(small, want if need(default) >= need(n) else binding.sdpa_kv(q, k, v, splits=default, tile=tile))
    # pages
    rows = 64
    blocks = -(-Skv // rows)
    pad = torch.zeros((B, Hkv, blocks * rows - Skv, D), dtype=k.dtype, device="cuda")
    pages = lambda t: torch.cat([t, pad], 2).view(B, Hkv, blocks, rows, D).transpose(1, 2).reshape(B * blocks, Hkv, rows, D).contiguous()
    table = torch.arange(B * blocks, dtype=torch.int32, device="cuda").view(B, blocks)
    lens = torch.full((B,), Skv, dtype=torch.int32, device="cuda")
    n = _count(binding, B, H, Hkv, Sq, blocks * rows, D, tile)
    args = (q, pages(k), pages(v), lens, table)
    assert torch.equal(binding.sdpa_paged(*args, tile=tile), binding.sdpa_paged(*args, tile=tile, splits=n))


def test_tiles_that_are_not_offered_are_refused_by_the_call():
    from paper_2603_01960_amd import binding
    q = torch.zeros((1, 2, 64, 64), dtype=torch.float16, device="cuda")
    for tile in ((32, 64), (64, 128), (256, 32), (64, 0)):
        with pytest.raises(binding.TiledSdpaError) as e:
            binding.sdpa_kv(q, q, q, tile=tile)
        assert e.value.status == 6
