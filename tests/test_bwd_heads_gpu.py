"""The backward of short sequences whose workgroups take one head after another (D = 64, 129 ... 256 rows, more than 256 heads;
csrc/sdpa_bwd_short_kernel.h): full and ragged last tiles, workgroups with one head, two and three, both masks, both types, against
float64; the first and the last 256 heads alone, a workgroup per head, give the same bits."""
import pytest
import torch

from test_bwd_forms_gpu import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,S", [(257, 256), (300, 129), (512, 160), (515, 161), (530, 225), (768, 197)])
def test_one_head_after_another(heads, S, causal):
    from paper_2603_01960_amd import binding
    for dtype, tol in ((torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)):       # times the gradient's size, as for every form
        g = torch.Generator("cuda").manual_seed(10 * S + heads)
        q, k, v, dout = (torch.randn((1, heads, S, 64), device="cuda", generator=g).to(dtype) for _ in range(4))
        o, lse = binding.sdpa(q, k, v, causal, return_lse=True)
        grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
        binding.sdpa_backward(q, k, v, o, dout, lse, causal, grads=grads)
        for h0 in (0, 255, heads - 1):            # a first head, the last of a round, the last of all
            for name, got, ref in zip(("dq", "dk", "dv"), grads, _reference(*(t[:, h0:h0 + 1] for t in (q, k, v, dout)), causal)):
                err = (got[:, h0:h0 + 1].double() - ref).abs().max().item()
                assert err <= tol * max(1.0, ref.abs().max().item()), f"{name} {dtype} head {h0} of {heads} S={S} causal={causal}: {err}"
        for h0 in (0, heads - 256):
            part = [t[:, h0:h0 + 256].contiguous() for t in (q, k, v, o, dout, lse)]
            alone = binding.sdpa_backward(*part, causal)
            assert all(torch.equal(a[:, h0:h0 + 256], b) for a, b in zip(grads, alone)), f"{dtype} heads {h0} ... S={S} causal={causal}"


@pytest.mark.parametrize("scale", [-0.125, 0.0, 0.5])
@pytest.mark.parametrize("causal", [False, True])
def test_scales(causal, scale):
    from paper_2603_01960_amd import binding
    heads, S = 530, 225
    for dtype, tol in ((torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)):
        g = torch.Generator("cuda").manual_seed(S)
        q, k, v, dout = (torch.randn((1, heads, S, 64), device="cuda", generator=g).to(dtype) for _ in range(4))
        o, lse = binding.sdpa(q, k, v, causal, scale, return_lse=True)
        grads = binding.sdpa_backward(q, k, v, o, dout, lse, causal, scale)
        for h0 in (0, heads - 1):
            for name, got, ref in zip(("dq", "dk", "dv"), grads, _reference(*(t[:, h0:h0 + 1] for t in (q, k, v, dout)), causal, scale)):
                err = (got[:, h0:h0 + 1].double() - ref).abs().max().item()
                assert err <= tol * max(1.0, ref.abs().max().item()), f"{name} {dtype} head {h0} scale={scale} causal={causal}: {err}"
