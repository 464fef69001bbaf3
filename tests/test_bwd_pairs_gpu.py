"""dK and dV at D = 160 come from pairs of wavefronts, the second of which works a tile behind the first: one to four pairs and
one or two streams per workgroup by the workgroups and the length of the chain of tiles.  Every form at one tile, an odd and an
even number of them, more streams than tiles, ragged ends and chains that run on into the next query head, against float64."""
import pytest
import torch

from test_bwd_forms_gpu import _reference

pytestmark = pytest.mark.gpu

# (key/value heads, query heads per key/value head, S)
CASES = [(1, 1, 1), (2, 1, 33), (1, 1, 64), (3, 1, 97), (9, 1, 160), (1, 3, 31), (2, 8, 45), (5, 4, 70), (40, 1, 225),       # one pair, two streams
         (90, 1, 129), (19, 1, 545), (38, 2, 300), (20, 8, 1090), (160, 8, 577),           # two pairs, two streams
         (260, 1, 40), (400, 1, 65), (170, 1, 200), (90, 4, 290), (210, 1, 385),            # two pairs, one stream
         (87, 1, 601), (64, 1, 897), (62, 2, 833)]                                          # four pairs (without the mask)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("hkv,G,S", CASES)
def test_gradients_of_pairs(hkv, G, S, dtype, causal):
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(100 * S + hkv)
    draw = lambda h: torch.randn((1, h, S, 160), device="cuda", generator=g).to(dtype)
    q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
    o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
    grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
    binding.sdpa_backward(q, k, v, o, dout, lse, causal, grads=grads)
    again = binding.sdpa_backward(q, k, v, o, dout, lse, causal)
    tol = 1.6e-2 if dtype == torch.bfloat16 else 2e-3      # times the gradient's size, as for every form of the backward pass
    for h in {0, hkv - 1}:
        hq = slice(h * G, (h + 1) * G)
        want = _reference(q[:, hq], k[:, h:h + 1], v[:, h:h + 1], dout[:, hq], causal)
        for name, got, ref in zip(("dq", "dk", "dv"), (grads[0][:, hq], grads[1][:, h:h + 1], grads[2][:, h:h + 1]), want):
            err = (got.double() - ref).abs().max().item()
            bound = tol * max(1.0, ref.abs().max().item())
            assert err <= bound, f"{name} heads={hkv}x{G} S={S} causal={causal}: {err} > {bound}"
    assert all(torch.isfinite(t).all() for t in grads)
    assert all(torch.equal(a, b) for a, b in zip(grads, again))       # no sum depends on who finishes first
