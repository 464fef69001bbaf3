"""The order in which workgroups take the tiles of a causal problem must not change what they compute (in the forward
pass not a single bit): each launch below is large enough for the long-tiles-first order (more than 256 workgroups) and is
held against calls that take the plain order (the linear-grid flag, or one head at a time).  Outputs start as NaN, so a tile nobody took shows."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _normal(*shape, dtype=torch.bfloat16, seed=0):
    g = torch.Generator("cuda").manual_seed(seed)
    return torch.randn(shape, device="cuda", generator=g).to(dtype)


# (B, H, S): one chunk of heads with a remainder of eight; several chunks, the first short; chunks of one head per XCD
# (K and V of a head beyond 8 MiB per eight heads); a ragged last tile
@pytest.mark.parametrize("B,H,S,D", [(1, 53, 640, 64), (5, 21, 600, 64), (3, 11, 8192, 128), (1, 3, 16500, 64), (7, 17, 333, 96),
                                     # 258, 301 and 512 workgroups: the second one of a CU in reverse order
                                     (1, 129, 200, 64), (1, 43, 850, 64), (1, 64, 1024, 160),
                                     # 513 ... 768 workgroups, up to three tiles per head: chunks of sixteen heads per XCD, a short
                                     # first one; two tiles of equal work: head after head; one tile per head: likewise
                                     (1, 231, 384, 64), (1, 257, 300, 96), (1, 256, 257, 128), (1, 300, 171, 96), (1, 257, 100, 64)])
def test_forward_order(B, H, S, D):
    from paper_2603_01960_amd import binding
    q, k, v = (_normal(B, H, S, D, seed=i) for i in range(3))
    out = torch.full_like(q, float("nan"))
    o = binding.sdpa(q, k, v, True, out=out)
    ref = binding.sdpa(q, k, v, True, flags=binding.FLAG_LINEAR_GRID)
    assert torch.equal(o, ref)


# folded query heads whose rows the 128-row tile divides, and does not; lengths that differ per batch entry
@pytest.mark.parametrize("B,H,Hkv,Sq,Skv,lens", [(3, 12, 3, 1024, 1024, None), (3, 24, 6, 333, 1000, None),
                                                 (5, 16, 8, 512, 1500, (1500, 0, 512, 777, 64)), (33, 16, 2, 1, 300, None)])
def test_cache_order(B, H, Hkv, Sq, Skv, lens):
    from paper_2603_01960_amd import binding
    D = 64
    q, k, v = _normal(B, H, Sq, D, seed=1), _normal(B, Hkv, Skv, D, seed=2), _normal(B, Hkv, Skv, D, seed=3)
    kv_lens = None if lens is None else torch.tensor(lens, dtype=torch.int32, device="cuda")
    out = torch.full_like(q, float("nan"))
    o = binding.sdpa_kv(q, k, v, True, out=out, kv_lens=kv_lens, splits=1, tile=(128, 64))
    for b in range(B):
        ref = binding.sdpa_kv(q[b:b + 1], k[b:b + 1], v[b:b + 1], True, splits=1, tile=(128, 64), flags=binding.FLAG_LINEAR_GRID,
                              kv_lens=None if lens is None else kv_lens[b:b + 1])
        # (a decoding step starts each head's sweep at a tile that depends on the workgroup: same sums, another order)
        if Sq == 1:
            assert (o[b].float() - ref[0].float()).abs().max() <= 1.6e-2
        else:
            assert torch.equal(o[b], ref[0])


@pytest.mark.parametrize("B,H,Hkv,S,D", [(1, 53, 53, 640, 64), (5, 24, 8, 600, 96), (9, 16, 16, 520, 128)])
def test_backward_order(B, H, Hkv, S, D):
    from paper_2603_01960_amd import binding
    q, k, v, dout = _normal(B, H, S, D, seed=1), _normal(B, Hkv, S, D, seed=2), _normal(B, Hkv, S, D, seed=3), _normal(B, H, S, D, seed=4)
    o, lse = binding.sdpa_kv(q, k, v, True, return_lse=True)
    grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    binding.sdpa_backward(q, k, v, o, dout, lse, True, grads=grads)
    G = H // Hkv
    for b in range(B):
        for h in range(0, Hkv, 3):
            hq = slice(h * G, (h + 1) * G)
            cut = lambda t, s: t[b:b + 1, s].contiguous()
            ref = binding.sdpa_backward(cut(q, hq), cut(k, slice(h, h + 1)), cut(v, slice(h, h + 1)), cut(o, hq), cut(dout, hq),
                                        cut(lse, hq), True)
            # a call on one head sums the same 16-bit products over tiles in another order (streams of tiles): FP32 sums that
            # differ by about 1e-6 of their largest terms, rounded to neighbouring BF16 values at most (2^-7 of the value)
            for got, want in ((grads[0][b, hq], ref[0][0]), (grads[1][b, h], ref[1][0, 0]), (grads[2][b, h], ref[2][0, 0])):
                got, want = got.float(), want.float()
                assert ((got - want).abs() <= want.abs() / 128 + 1e-4 * want.abs().max()).all()
    assert all(torch.isfinite(t.float()).all() for t in grads)
