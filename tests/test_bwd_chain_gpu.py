"""The backward pass in five products, whose dQ is summed from block to block of 256 keys (csrc/sdpa_bwd_chain_kernel.h): ragged ends of
tiles and blocks, one and several rounds of blocks, heads that eight does not divide, grouped heads, both masks, both
types, against float64; a second call gives the same bits, and a workspace of the least size the passes that need no sums."""
import pytest
import torch

from test_bwd_forms_gpu import CASES as FORMS
from test_bwd_forms_gpu import _reference
from test_bwd_joint_gpu import CASES as JOINT

pytestmark = pytest.mark.gpu

# (D, key/value heads, query heads per key/value head, S, causal)
CASES = [(64, 128, 1, 2048, False), (64, 62, 1, 2041, False), (64, 32, 4, 2048, False), (64, 32, 1, 4096, True), (64, 16, 1, 8170, True),
         (96, 64, 1, 2048, False), (96, 64, 2, 1000, False), (96, 31, 1, 3999, True), (96, 32, 3, 4070, True), (96, 24, 1, 5100, False),
         (128, 64, 1, 1024, False), (128, 62, 1, 2041, False), (128, 64, 3, 1000, False), (128, 64, 1, 2048, True), (128, 62, 1, 2017, True),
         (128, 16, 1, 8129, False), (128, 15, 1, 8190, True), (128, 32, 2, 4095, True),
         # one block of keys, nothing to sum
         (128, 256, 8, 256, False),
         # a last block whose queries are one tile, full and ragged, alone and with the next query head behind it
         (128, 64, 1, 4128, True), (128, 64, 1, 4097, True), (128, 64, 2, 4097, True), (96, 31, 1, 4110, True), (64, 16, 1, 8200, True),
         # the end of the keys inside a block without a ragged tile; the diagonal's last block with two, four, six tiles
         (64, 62, 1, 2016, False), (128, 32, 1, 4064, False), (64, 16, 1, 8256, True), (128, 64, 1, 2240, True), (96, 32, 1, 4000, True)]


@pytest.mark.parametrize("D,hkv,G,S,causal", CASES)
def test_gradients_summed_from_block_to_block(D, hkv, G, S, causal):
    from paper_2603_01960_amd import binding
    full, least = binding.bwd_full_workspace_bytes(1, hkv * G, hkv, S, D, causal), binding.bwd_workspace_bytes(1, hkv * G, S)
    assert full > least                           # else the call takes other kernels
    for dtype, tol in ((torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)):       # times the gradient's size, as for every form
        g = torch.Generator("cuda").manual_seed(100 * S + hkv)
        draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
        q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
        o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
        grads = tuple(torch.full_like(t, float("nan")) for t in (q, k, v))
        workspace = torch.full((-(-full // 4),), -1, dtype=torch.int32, device="cuda")     # (nothing in it is taken for zero)
        binding.sdpa_backward(q, k, v, o, dout, lse, causal, grads=grads, workspace=workspace)
        again = binding.sdpa_backward(q, k, v, o, dout, lse, causal)
        passes = binding.sdpa_backward(q, k, v, o, dout, lse, causal, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
        for h in {0, hkv - 1}:
            hq = slice(h * G, (h + 1) * G)
            want = _reference(q[:, hq], k[:, h:h + 1], v[:, h:h + 1], dout[:, hq], causal)
            for name, got, other, ref in zip(("dq", "dk", "dv"), (grads[0][:, hq], grads[1][:, h:h + 1], grads[2][:, h:h + 1]),
                                             (passes[0][:, hq], passes[1][:, h:h + 1], passes[2][:, h:h + 1]), want):
                err = (got.double() - ref).abs().max().item()
                bound = tol * max(1.0, ref.abs().max().item())
                assert err <= bound, f"{name} {dtype} heads={hkv}x{G} S={S} causal={causal}: {err} > {bound}"
                # no less precise than the passes: both round dS and P once to 16 bits and sum in FP32 (2-norm, 2 % for the order)
                assert (got.double() - ref).norm() <= 1.02 * (other.double() - ref).norm(), f"{name} {dtype}"
        assert all(torch.isfinite(t).all() for t in grads)
        assert all(torch.equal(a, b) for a, b in zip(grads, again))   # no sum depends on who finishes first


@pytest.mark.parametrize("dtype,tol", [(torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)])
def test_passes_where_the_workspace_has_no_room_for_the_sums(dtype, tol):
    """The cases of the passes that take the five products when torch allocates the workspace, with one of the least size."""
    from paper_2603_01960_amd import binding
    taken = 0
    for causal in (False, True):
        for D, hkv, G, S in [*JOINT, *((D, *c) for D in (64, 96, 128) for c in FORMS)]:
            least = binding.bwd_workspace_bytes(1, hkv * G, S)
            if binding.bwd_full_workspace_bytes(1, hkv * G, hkv, S, D, causal) == least:
                continue
            taken += 1
            g = torch.Generator("cuda").manual_seed(S + hkv)
            draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
            q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
            o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
            grads = binding.sdpa_backward(q, k, v, o, dout, lse, causal, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
            want = _reference(q[:, -G:], k[:, -1:], v[:, -1:], dout[:, -G:], causal)
            for name, got, ref in zip(("dq", "dk", "dv"), (grads[0][:, -G:], grads[1][:, -1:], grads[2][:, -1:]), want):
                err = (got.double() - ref).abs().max().item()
                assert err <= tol * max(1.0, ref.abs().max().item()), f"{name} D={D} heads={hkv}x{G} S={S} causal={causal}: {err}"
    assert taken > 0


@pytest.mark.parametrize("scale", [-0.125, 0.0, 0.5])
@pytest.mark.parametrize("D,hkv,G,S,causal", [(64, 62, 1, 2041, False), (64, 16, 1, 8170, True), (96, 31, 1, 3999, True), (128, 32, 2, 4095, True)])
def test_scales(D, hkv, G, S, causal, scale):
    """The sign of a scale, which the scores take with their factor here and with an operand in the statistics; none at all; and one under which
    a few keys have most of a row's weight."""
    from paper_2603_01960_amd import binding
    assert binding.bwd_full_workspace_bytes(1, hkv * G, hkv, S, D, causal) > binding.bwd_workspace_bytes(1, hkv * G, S)
    for dtype, tol in ((torch.float16, 2e-3), (torch.bfloat16, 1.6e-2)):
        g = torch.Generator("cuda").manual_seed(S + D)
        draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
        q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
        o, lse = binding.sdpa_kv(q, k, v, causal, scale=scale, return_lse=True)
        grads = binding.sdpa_backward(q, k, v, o, dout, lse, causal, scale)
        least = torch.empty(binding.bwd_workspace_bytes(1, hkv * G, S), dtype=torch.uint8, device="cuda")
        passes = binding.sdpa_backward(q, k, v, o, dout, lse, causal, scale, workspace=least)
        last = lambda t: (t[0][:, -G:], t[1][:, -1:], t[2][:, -1:])
        want = _reference(q[:, -G:], k[:, -1:], v[:, -1:], dout[:, -G:], causal, scale)
        for name, got, other, ref in zip(("dq", "dk", "dv"), last(grads), last(passes), want):
            err = (got.double() - ref).abs().max().item()
            bound = tol * max(1.0, ref.abs().max().item())
            assert err <= bound, f"{name} {dtype} scale={scale}: {err} > {bound}"
            assert (got.double() - ref).norm() <= 1.02 * (other.double() - ref).norm(), f"{name} {dtype} scale={scale}"


def test_passes_where_torch_has_no_memory_for_the_sums():
    """With less memory left than the sums need, but enough for the statistics, the call gives what a workspace of the least size does."""
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(7)
    q, k, v, dout = (torch.randn((2, 64, 2048, 128), device="cuda", generator=g).bfloat16() for _ in range(4))
    o, lse = binding.sdpa(q, k, v, True, return_lse=True)
    full, least = binding.bwd_full_workspace_bytes(2, 64, 64, 2048, 128, True), binding.bwd_workspace_bytes(2, 64, 2048)
    assert full > 128 << 20 and least < 16 << 20
    want = binding.sdpa_backward(q, k, v, o, dout, lse, True, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    sums = binding.sdpa_backward(q, k, v, o, dout, lse, True)
    grads = tuple(torch.empty_like(t) for t in (q, k, v))
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(full, dtype=torch.uint8, device="cuda")
        binding.sdpa_backward(q, k, v, o, dout, lse, True, grads=grads)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert all(torch.equal(a, b) for a, b in zip(grads, want))
    assert not all(torch.equal(a, b) for a, b in zip(grads, sums))       # (so it was the other form)


@pytest.mark.parametrize("dtype,tol", [(torch.float16, 4e-3), (torch.bfloat16, 3.2e-2)])          # twice that of each form to float64
@pytest.mark.parametrize("D,hkv,G,S,causal", [(64, 62, 1, 2041, False), (96, 31, 1, 3999, True), (128, 62, 1, 2041, False), (128, 32, 2, 4095, True)])
def test_keys_of_infinities(D, hkv, G, S, causal, dtype, tol):
    """A key whose score is -inf for every query has gradients of zero, also where rows past the end, whose score with it is NaN (0 * inf),
    lie in the last tile.  dQ is NaN in its column, 0 * inf, of the rows that see it and, under the mask, ahead of it in its tile, and nowhere
    else."""
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(S + D)
    draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).to(dtype)
    q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
    q[..., 0] = q[..., 0].abs() + 0.1
    keys = [S // 2, S - 300]
    k[0, hkv - 1, keys, 0] = float("-inf")
    o, lse = binding.sdpa_kv(q, k, v, causal, return_lse=True)
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()
    assert binding.bwd_full_workspace_bytes(1, hkv * G, hkv, S, D, causal) > binding.bwd_workspace_bytes(1, hkv * G, S)
    grads = binding.sdpa_backward(q, k, v, o, dout, lse, causal)
    passes = binding.sdpa_backward(q, k, v, o, dout, lse, causal,
                                   workspace=torch.empty(binding.bwd_workspace_bytes(1, hkv * G, S), dtype=torch.uint8, device="cuda"))
    spoilt = torch.zeros(grads[0].shape, dtype=torch.bool, device="cuda")
    spoilt[0, -G:, keys[0] // 32 * 32 if causal else 0:, 0] = True
    assert torch.equal(torch.isnan(grads[0]), spoilt)
    for name, got, ref in zip(("dq", "dk", "dv"), grads, passes):
        assert torch.isfinite(got[..., 1:]).all() and torch.isfinite(ref[..., 1:]).all(), name
        assert name == "dq" or (torch.isfinite(got).all() and torch.isfinite(ref).all()), name
        both = torch.isfinite(got) & torch.isfinite(ref)
        assert (got[both] - ref[both]).abs().max() <= tol * max(1.0, ref[both].abs().max()), name
    assert (grads[1][0, hkv - 1, keys] == 0).all() and (grads[2][0, hkv - 1, keys] == 0).all()


def test_workspace_that_begins_in_the_middle_of_a_cache_line():
    """A workspace needs no more than 16 bytes of alignment; the sums then still keep to cache lines of their own."""
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(6)
    q, k, v, dout = (torch.randn((1, 64, 2048, 128), device="cuda", generator=g).bfloat16() for _ in range(4))
    o, lse = binding.sdpa(q, k, v, True, return_lse=True)
    full = binding.bwd_full_workspace_bytes(1, 64, 64, 2048, 128, True)
    room = torch.full((full + 512,), 255, dtype=torch.uint8, device="cuda")
    base = -room.data_ptr() % 256
    want = binding.sdpa_backward(q, k, v, o, dout, lse, True, workspace=room[base:base + full])
    for shift in (16, 112, 240):
        room.fill_(255)
        got = binding.sdpa_backward(q, k, v, o, dout, lse, True, workspace=room[base + shift:base + shift + full])
        assert all(torch.equal(a, b) for a, b in zip(want, got)), f"begins {shift} bytes into a line"
        assert (room[:base + shift] == 255).all() and (room[base + shift + full:] == 255).all()


def test_recorded_into_a_graph_and_on_two_streams():
    """The counters of a call are cleared by a kernel of its own: every replay, and two calls under way at once, give the eager bits."""
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(5)
    q, k, v, dout = (torch.randn((1, 64, 2048, 128), device="cuda", generator=g).bfloat16() for _ in range(4))
    o, lse = binding.sdpa(q, k, v, True, return_lse=True)
    full = binding.bwd_full_workspace_bytes(1, 64, 64, 2048, 128, True)
    assert full > binding.bwd_workspace_bytes(1, 64, 2048)
    want = binding.sdpa_backward(q, k, v, o, dout, lse, True)
    sets = [(torch.full((full,), 255, dtype=torch.uint8, device="cuda"), tuple(torch.empty_like(t) for t in (q, k, v))) for _ in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in sets]
    for _ in range(3):
        for (workspace, grads), stream in zip(sets, streams):
            with torch.cuda.stream(stream):
                binding.sdpa_backward(q, k, v, o, dout, lse, True, workspace=workspace, grads=grads)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for _, grads in sets for a, b in zip(grads, want))
    workspace, grads = sets[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.sdpa_backward(q, k, v, o, dout, lse, True, workspace=workspace, grads=grads)
    for _ in range(4):
        for t in grads:
            t.fill_(float("nan"))
        workspace.fill_(170)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(grads, want))


@pytest.mark.parametrize("D,hkv,G,S", [(64, 16, 1, 8170), (96, 31, 1, 3999), (96, 32, 3, 4070), (128, 64, 1, 2048), (128, 62, 1, 2017), (128, 32, 2, 4095)])
def test_rows_of_nan_stay_with_the_keys_they_see(D, hkv, G, S):
    """Under the mask a query row that is not finite, in Q (with O and LSE) or in dO, changes nothing for the keys behind its tile of 32, nor
    for the other query rows that come before it or belong to other heads."""
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(S - D)
    draw = lambda h: torch.randn((1, h, S, D), device="cuda", generator=g).bfloat16()
    q, k, v, dout = draw(hkv * G), draw(hkv), draw(hkv), draw(hkv * G)
    assert binding.bwd_full_workspace_bytes(1, hkv * G, hkv, S, D, True) > binding.bwd_workspace_bytes(1, hkv * G, S)
    o, lse = binding.sdpa_kv(q, k, v, True, return_lse=True)
    want = binding.sdpa_backward(q, k, v, o, dout, lse, True)
    last = hkv * G - 1
    # a first block's first tile and its last one, a wavefront's second 32 keys, tiles of the last block
    for row in (5, 255, 1067, S - 200, S - 1):
        for where in ("q", "dout"):
            q1, d1 = q.clone(), dout.clone()
            (q1 if where == "q" else d1)[0, last, row] = float("nan")
            o1, lse1 = binding.sdpa_kv(q1, k, v, True, return_lse=True) if where == "q" else (o, lse)
            dq, dk, dv = binding.sdpa_backward(q1, k, v, o1, d1, lse1, True)
            behind = (row // 32 + 1) * 32
            assert torch.isnan(dv[0, -1, :row + 1]).all()
            assert torch.equal(dk[0, -1, behind:], want[1][0, -1, behind:]), f"dk, {where} row {row}"
            assert torch.equal(dv[0, -1, behind:], want[2][0, -1, behind:]), f"dv, {where} row {row}"
            assert torch.equal(dk[0, :-1], want[1][0, :-1]) and torch.equal(dv[0, :-1], want[2][0, :-1])
            others = torch.arange(S, device="cuda") != row
            assert torch.equal(dq[0, last, others], want[0][0, last, others]), f"dq, {where} row {row}"
            assert torch.equal(dq[0, :last], want[0][0, :last])
