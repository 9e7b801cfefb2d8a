"""Batches whose matrices pass 32-bit offsets: 36 million samples of a small model."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wd", ["f32", "bf16"])
def test_large_batch(wd):
    """The gradient with all but a few coefficients zero, and log pi of the same samples, against the call on those alone:
    the same products, in another order of the ks (2^-24 a rounding, sums of up to 24 or 300 terms: 1e-5; a flip of a BF16
    rounding in relu(A) or an adjoint: 2^-8 of a term)."""
    from paper_2106_13308_amd import binding as Bd, inputs

    n, h, B = 20, 24, 36_000_037
    rtol = 1e-5 if wd == "f32" else 2.0 ** -8
    p = inputs.made_init(n, h, 5)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.F32 if wd == "f32" else Bd.BF16, band=False)
    g = torch.Generator(device="cuda").manual_seed(1)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8, device="cuda")
    pick = torch.cat([torch.arange(0, 100), torch.arange(B // 2, B // 2 + 100), torch.arange(B - 100, B)]).cuda()
    few = S[:300].clone()
    few[:, :n] = 2 * torch.randint(0, 2, (300, n), generator=g, device="cuda", dtype=torch.int8) - 1
    S[:, :n] = 1
    S[pick] = few
    coef = torch.zeros(B, device="cuda")
    coef[pick] = cf = torch.randn(300, generator=g, device="cuda")
    lp, ref = Bd.logprob(m, S), Bd.logprob(m, few)
    assert (lp[pick] - ref).abs().max() <= rtol * ref.abs().max()
    got = Bd.logprob_backward(m, S, coef)
    for a, b in zip(got, Bd.logprob_backward(m, few, cf)):
        assert (a - b).abs().max() <= 4 * rtol * b.abs().max()
