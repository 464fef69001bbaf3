"""Buffers that a caller passes for the kernels to write to: refused before any launch unless they are on the device of the
call and one range of bytes; taken where they are, whatever their shape."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(n=4):
    g = torch.Generator("cuda").manual_seed(1)
    return [torch.randn((1, 2, 64, 64), device="cuda", generator=g).half() for _ in range(n)]


def test_workspaces_on_the_host_or_with_gaps_are_refused():
    from paper_2603_01960_amd import binding
    q, k, v, dout = _tensors()
    lens = torch.full((1,), 64, dtype=torch.int32, device="cuda")
    table = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    o, lse = binding.sdpa(q, k, v, return_lse=True)
    need = max(binding.kv_workspace_bytes(1, 2, 64, 64, 2), binding.bwd_workspace_bytes(1, 2, 64))
    calls = {"kv": lambda w: binding.sdpa_kv(q, k, v, splits=2, workspace=w),
             "paged": lambda w: binding.sdpa_paged(q, k, v, lens, table, splits=2, workspace=w),
             "backward": lambda w: binding.sdpa_backward(q, k, v, o, dout, lse, workspace=w)}
    byte = dict(dtype=torch.uint8)
    for call in calls.values():
        for bad in (torch.empty(need, **byte), torch.empty(2 * need, device="cuda", **byte)[::2],
                    torch.empty(1, device="cuda", **byte).expand(need), torch.empty((need, 2), device="cuda", **byte)[:, 0]):
            with pytest.raises(ValueError, match="workspace"):
                call(bad)
    # one range of bytes in any shape, order or type
    want = {name: call(None) for name, call in calls.items()}
    for good in (torch.empty(need, device="cuda", **byte), torch.empty((4, need), device="cuda", **byte).t(),
                 torch.empty(need, device="cuda", dtype=torch.float32)):
        for name, call in calls.items():
            got = call(good)
            for a, b in zip(got if name == "backward" else (got,), want[name] if name == "backward" else (want[name],)):
                assert torch.equal(a, b)
    # (not looked at where the call needs none)
    assert torch.isfinite(binding.sdpa_kv(q, k, v, splits=1, workspace=torch.empty(1, **byte)).float()).all()


def test_lse_out_on_the_host_is_refused():
    from paper_2603_01960_amd import binding
    q, k, v = _tensors(3)
    with pytest.raises(ValueError, match="lse_out"):
        binding.sdpa(q, k, v, return_lse=True, lse_out=torch.empty((1, 2, 64)))
    lse = torch.empty((1, 2, 64), device="cuda")
    assert binding.sdpa(q, k, v, return_lse=True, lse_out=lse)[1] is lse
