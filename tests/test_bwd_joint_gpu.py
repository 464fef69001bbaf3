"""The backward pass in one grid for dQ and dK + dV, and its dK + dV pass by pairs of wavefronts at D = 160: every form of either
(wavefronts along the rows and streams of both passes, by the workgroups and the length of their chains of tiles), and the
passes in launches of their own, with one tile, odd and even numbers of them, more streams than tiles, ragged ends
and chains that run on into the next query head, against float64."""
import pytest
import torch

from test_bwd_forms_gpu import _reference

pytestmark = pytest.mark.gpu

# (D, key/value heads, query heads per key/value head, S)
CASES = [(64, 1, 1, 257), (64, 3, 1, 300), (64, 45, 1, 290), (64, 48, 1, 300),            # 32 keys and four streams; 128 keys
         (64, 310, 1, 290), (64, 320, 1, 300), (64, 6, 1, 1030), (64, 4, 1, 1000),         # ... the passes apart; long chains
         (64, 1, 4, 1), (64, 2, 8, 31), (64, 1, 8, 330), (64, 3, 5, 513), (64, 33, 4, 200), (64, 70, 2, 129),
         (96, 5, 1, 65), (96, 22, 1, 225), (96, 40, 1, 97), (96, 24, 1, 520), (96, 48, 1, 390), (96, 25, 1, 2050), (96, 110, 1, 290),
         (96, 6, 1, 1100), (96, 2, 1, 3500), (96, 9, 1, 993),
         (96, 3, 4, 33), (96, 44, 3, 70), (96, 12, 3, 449), (96, 40, 8, 1770), (96, 250, 4, 290),
         (128, 3, 1, 40), (128, 40, 1, 90), (128, 20, 1, 193), (128, 7, 1, 450), (128, 130, 1, 200), (128, 11, 1, 900), (128, 30, 1, 800),
         (128, 40, 1, 481), (128, 1, 8, 17), (128, 4, 3, 290), (128, 10, 8, 801), (128, 56, 8, 801), (128, 50, 2, 300),
         # D = 160: one pair and two streams, two pairs and two streams, two pairs, four pairs
         (160, 1, 1, 65), (160, 3, 1, 97), (160, 9, 1, 160), (160, 1, 3, 31), (160, 2, 8, 45), (160, 5, 4, 70), (160, 90, 4, 145),
         (160, 20, 3, 300), (160, 26, 8, 257), (160, 30, 2, 290), (160, 19, 3, 545), (160, 30, 8, 1090),
         (160, 1, 1, 1), (160, 2, 1, 33), (160, 260, 1, 40), (160, 90, 1, 129), (160, 400, 1, 65), (160, 120, 2, 150),
         (160, 64, 1, 897), (160, 90, 4, 290), (160, 210, 1, 385), (160, 210, 1, 601),
         # passes in launches of their own, in every form of either, and what else the lines above leave out: test_bwd_pick_host.py
         # finds the kernels that some call takes and no case meets
         (64, 15, 2, 2564), (96, 17, 2, 130), (96, 260, 1, 130), (96, 22, 1, 680), (96, 4, 1, 1923), (96, 13, 1, 1154), (96, 5, 2, 770),
         (96, 112, 1, 67), (128, 17, 2, 129), (128, 134, 4, 33), (128, 86, 1, 1037), (128, 2, 1, 5601), (128, 15, 1, 1158), (128, 16, 4, 1024),
         (128, 32, 2, 2040), (96, 12, 1, 964), (96, 203, 1, 129)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D,hkv,G,S", CASES)
def test_gradients_of_one_grid(D, hkv, G, S, causal):
    from paper_2603_01960_amd import binding
    for dtype, tol in ((torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)):       # times the gradient's size, as for every form
        g = torch.Generator("cuda").manual_seed(100 * S + hkv)
        draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
        q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
        o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
        grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
        binding.sdpa_backward(q, k, v, o, dout, lse, causal, grads=grads)
        again = binding.sdpa_backward(q, k, v, o, dout, lse, causal)
        for h in {0, hkv - 1}:
            hq = slice(h * G, (h + 1) * G)
            want = _reference(q[:, hq], k[:, h:h + 1], v[:, h:h + 1], dout[:, hq], causal)
            for name, got, ref in zip(("dq", "dk", "dv"), (grads[0][:, hq], grads[1][:, h:h + 1], grads[2][:, h:h + 1]), want):
                err = (got.double() - ref).abs().max().item()
                bound = tol * max(1.0, ref.abs().max().item())
                assert err <= bound, f"{name} {dtype} heads={hkv}x{G} S={S} causal={causal}: {err} > {bound}"
        assert all(torch.isfinite(t).all() for t in grads)
        assert all(torch.equal(a, b) for a, b in zip(grads, again))   # no sum depends on who finishes first
