"""Scores of -infinity, which finite BF16 operands reach through an overflowing product: such keys have weight 0 wherever
they lie -- ahead of a row's other keys, filling a tile, a stream of tiles or a whole split -- and only a row without any
finite score has no value (NaN).  Every form of the forward pass, against softmax in float64."""
import pytest
import torch

pytestmark = pytest.mark.gpu

BIG = 1e30                                        # BIG * BIG overflows float32

# (heads, Sq, Skv, D, splits); Sq == Skv: the square entry point.  Streams of the square problem, its plain form; the decoding
# kernel in one run, in runs it combines itself, in runs for the merge kernel; streams against a cache, alone and split;
# long query blocks with many splits and rows
FORMS = [(4, 1024, 1024, 64, 0), (3, 700, 700, 128, 0), (500, 300, 300, 64, 0), (9, 1000, 1000, 96, 0),
         (200, 1, 700, 128, 0), (8, 4, 700, 128, 4), (8, 4, 2000, 64, 40), (3, 20, 900, 160, 3),
         (4, 40, 2000, 128, 1), (4, 40, 2000, 64, 3), (300, 200, 700, 64, 2), (9, 300, 700, 96, 3)]


def _expected(q, k, v):
    s = (q.double() @ k.double().t().contiguous()).float().double()            # overflows where the kernel's sums do
    return (s * q.shape[-1] ** -0.5).softmax(-1) @ v.double()


@pytest.mark.parametrize("heads,Sq,Skv,D,splits", FORMS)
def test_keys_of_infinitely_low_score_have_no_weight(heads, Sq, Skv, D, splits):
    from paper_2603_01960_amd import binding
    g = torch.Generator("cuda").manual_seed(heads + Sq)
    q, k, v = (torch.randn((1, heads, n, D), device="cuda", generator=g).bfloat16() for n in (Sq, Skv, Skv))
    row, h = Sq // 2, heads // 2
    # dimension 0 gives the score to keys of one row's choice, and nothing to anyone else
    q[..., 0] = 0
    k[..., 0] = 0
    q[0, h, row, 0] = BIG
    call = (lambda: binding.sdpa(q, k, v)) if Sq == Skv else (lambda: binding.sdpa_kv(q, k, v, splits=splits))
    plain = call()
    nan = torch.zeros((1, heads, Sq), dtype=torch.bool, device="cuda")
    for low in (range(32, 64), range(0, 32), range(96, 224), range(0, Skv // 2), range(Skv // 2, Skv), range(1, Skv)):
        k[0, h, :, 0] = 0
        k[0, h, low.start:low.stop, 0] = -BIG
        out = call()
        want = _expected(q[0, h], k[0, h], v[0, h])
        assert (out[0, h].double() - want).abs().max().item() <= 1.6e-2, low
        keep = torch.arange(heads, device="cuda") != h
        assert torch.equal(out[:, keep], plain[:, keep])
    # nothing but -inf: no value for that row, all others as before
    k[0, h, :, 0] = -BIG
    out = call()
    nan[0, h, row] = True
    assert torch.equal(out.isnan().all(-1), nan) and torch.equal(out.isnan().any(-1), nan)


def test_rows_without_keys_are_still_told_apart():
    """O = 0 and LSE = -inf where no key reaches a row, NaN only where keys do: under the causal mask with an entry shorter than
    the query block, in every form a cache call takes."""
    from paper_2603_01960_amd import binding
    for Sq, D, splits in ((4, 128, 1), (4, 128, 4), (4, 64, 40), (40, 64, 1), (40, 64, 3), (200, 96, 2)):
        q, k, v = (torch.randn((2, 2, n, D), device="cuda").bfloat16() for n in (Sq, 1000, 1000))
        q[..., 0], k[..., 0] = 0, 0
        q[1, 1, Sq - 1, 0] = BIG
        k[1, 1, :, 0] = -BIG
        lens = torch.tensor([Sq - 2, Sq - 1], dtype=torch.int32, device="cuda")
        o, lse = binding.sdpa_kv(q, k, v, True, kv_lens=lens, splits=splits, return_lse=True)
        assert (o[0, :, :2] == 0).all() and (o[1, :, :1] == 0).all()
        assert (lse[0, :, :2] == -float("inf")).all() and (lse[1, :, :1] == -float("inf")).all()
        assert o[1, 1, Sq - 1].isnan().all() and o.isnan().sum() == D
        assert torch.isfinite(lse[0, :, 2:]).all()
