"""The square forward pass splits its K/V tiles over up to eight streams per workgroup where the workgroups are few, and the
number of streams and of query rows follows from the head dim, the mask, the workgroups and the length of the chain of
tiles: every form at lengths around its tiles (32 keys, 32 to 128 rows) and with fewer tiles than streams, against float64 on
the same inputs: the usual forward tolerances."""
import pytest
import torch

pytestmark = pytest.mark.gpu

# (heads, S): at most 64, 128, 256, 320 and 400 workgroups of 128 rows on short, medium and long chains; two tiles; odd tails
CASES = [(1, 33), (3, 64), (2, 65), (2, 96), (1, 97), (5, 129), (4, 300), (2, 2049), (70, 130), (70, 200), (25, 520), (13, 1030), (5, 2500),
         (80, 255), (40, 515), (25, 1025), (10, 2100), (12, 2300), (40, 1024), (24, 2048), (9, 4100), (60, 64)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("D", [64, 96, 128, 160])
def test_outputs_of_every_form(D, causal):
    from paper_2603_01960_amd import binding
    for i, (H, S) in enumerate(CASES):
        dtype = torch.bfloat16 if i % 2 else torch.float16
        g = torch.Generator("cuda").manual_seed(8000 + i)
        q, k, v = (torch.randn((1, H, S, D), device="cuda", generator=g).to(dtype) for _ in range(3))
        out, lse_out = torch.full_like(q, float("nan")), torch.full((1, H, S), float("nan"), device="cuda")
        binding.sdpa(q, k, v, causal, return_lse=True, out=out, lse_out=lse_out)
        tol = 1.6e-2 if dtype == torch.bfloat16 else 2e-3
        assert torch.isfinite(out.float()).all() and torch.isfinite(lse_out).all()
        for h in {0, H // 2, H - 1}:
            qd, kd, vd = (t[0, h].double() for t in (q, k, v))
            s = (qd @ kd.t().contiguous()) * D ** -0.5
            if causal:
                s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
            err = (out[0, h].double() - s.softmax(-1) @ vd).abs().max().item()
            lerr = (lse_out[0, h].double() - s.logsumexp(-1)).abs().max().item()
            assert err <= tol and lerr <= 1e-4, f"D={D} heads={H} S={S} causal={causal}: {err}, lse {lerr}"
        # a NaN query row stays NaN and alone
        if i % 4 == 0:
            q[0, 0, S // 2, 3] = float("nan")
            o = binding.sdpa(q, k, v, causal)
            assert o[0, 0, S // 2].isnan().all() and o.isnan().sum() == D
