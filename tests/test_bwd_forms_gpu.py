"""The backward pass at lengths around its tiles (32 streamed rows, 32 to 128 resident ones), with fewer tiles than streams, few and
many workgroups, short and long chains of tiles and grouped heads, against float64 gradients.  Which kernels the cases meet follows
from pick_bwd_joint and pick_bwd_form (csrc/sdpa_bwd_pick.h); together with those of test_bwd_joint_gpu.py they meet every one that
some call takes (test_bwd_pick_host.py)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reference(q, k, v, dout, causal, scale=None):
    """Gradients of Eq. 1 in float64; k and v repeated over the heads of a group, their gradients summed."""
    G = q.shape[1] // k.shape[1]
    q, dout = q.double(), dout.double()
    kr, vr = (t.double().repeat_interleave(G, 1) for t in (k, v))
    scale = q.shape[-1] ** -0.5 if scale is None else scale
    s = (q @ kr.transpose(2, 3).contiguous()) * scale
    if causal:
        s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    p = s.softmax(-1)
    dp = dout @ vr.transpose(2, 3).contiguous()
    ds = p * (dp - (p * dp).sum(-1, keepdim=True))
    fold = lambda t: t.view(t.shape[0], -1, G, *t.shape[2:]).sum(2)
    return (ds @ kr) * scale, fold(ds.transpose(2, 3).contiguous() @ q) * scale, fold(p.transpose(2, 3).contiguous() @ dout)


# (B * Hkv, G, S): at most 64, 128, 256 and 400 workgroups of 128 rows on short, medium and long chains; more streams than tiles;
# chains that continue into the next query head of a group
CASES = [(1, 1, 65), (3, 1, 96), (2, 1, 97), (5, 1, 300), (2, 1, 2049), (1, 8, 33), (3, 4, 70), (2, 3, 161), (70, 1, 200), (24, 1, 520),
         # whole heads in one workgroup (D = 64, 96): one to eight 32-row blocks, full and ragged
         (3, 1, 1), (2, 1, 16), (5, 1, 32), (4, 1, 33), (2, 1, 64), (3, 1, 100), (2, 1, 128), (130, 1, 129), (120, 1, 160), (256, 1, 197),
         (112, 1, 224), (115, 1, 255), (111, 1, 256),
         (7, 1, 2100), (35, 2, 257), (45, 1, 515), (25, 1, 1030), (16, 4, 513), (13, 1, 2050), (20, 1, 2048),
         # many workgroups of grouped heads, the tiles of a group's heads one head after the other: odd and even tile counts, full and
         # ragged
         (105, 2, 513), (140, 3, 300), (135, 2, 384), (205, 4, 160), (64, 2, 1024), (66, 2, 1100)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 96, 128, 160])
def test_gradients_of_every_form(D, causal):
    from paper_2603_01960_amd import binding
    for i, (hkv, G, S) in enumerate(CASES):
        dtype = torch.bfloat16 if i % 2 else torch.float16
        g = torch.Generator("cuda").manual_seed(7000 + i)
        draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
        q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
        o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
        grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
        binding.sdpa_backward(q, k, v, o, dout, lse, causal, grads=grads)
        again = binding.sdpa_backward(q, k, v, o, dout, lse, causal)
        tol = 1.6e-2 if dtype == torch.bfloat16 else 2e-3
        # the first and the last key/value head with their query heads
        for h in {0, hkv - 1}:
            hq = slice(h * G, (h + 1) * G)
            want = _reference(q[:, hq], k[:, h:h + 1], v[:, h:h + 1], dout[:, hq], causal)
            for name, got, ref in zip(("dq", "dk", "dv"), (grads[0][:, hq], grads[1][:, h:h + 1], grads[2][:, h:h + 1]), want):
                err = (got.double() - ref).abs().max().item()
                bound = tol * max(1.0, ref.abs().max().item())
                assert err <= bound, f"{name} D={D} heads={hkv}x{G} S={S} causal={causal}: {err} > {bound}"
        for a, b in zip(grads, again):
            assert torch.equal(a, b)              # no sum depends on who finishes first
