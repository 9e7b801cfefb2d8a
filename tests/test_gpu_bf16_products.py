"""The BF16 products at the edges of their tiles, stages and staircases, against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one entry each; one more or less than a 64-tile and a 64-column stage; an odd and an even number of
# 32-column steps; the 128 x 128 shapes of the adjoint (512 of them) and of the weight gradient (more than
# 64); staircases that jump over many units or sites at once
SHAPES = [(2, 1, 1, "default"), (64, 64, 64, "default"), (65, 63, 65, "default"), (97, 33, 31, "default"),
          (129, 257, 190, "default"), (40, 900, 70, "default"), (900, 40, 130, "default"), (300, 300, 100, "all_first"),
          (300, 300, 100, "all_last"), (1300, 700, 66, "clustered"), (70, 2049, 4097, "default"), (1100, 1030, 70, "default")]


def _degrees(kind, n, h):
    from paper_2106_13308_amd import inputs

    if kind == "all_first":
        return np.ones(h, np.int32)
    if kind == "all_last":
        return np.full(h, n - 1, np.int32)
    if kind == "clustered":  # bursts of units at three sites
        return np.sort(np.random.default_rng(4).choice([1, n // 3, n - 2], size=h)).astype(np.int32)
    return inputs.made_degrees(n, h)


@pytest.mark.parametrize("n,h,B,kind", SHAPES)
def test_bf16_products(n, h, B, kind):
    """log pi within 2e-2 of its size, the logits' BF16 bar, and the gradient of sum_b coef_b log pi within 3e-2 of
    each array's largest entry (three BF16 roundings of 2^-8 between the weights and an entry)."""
    from oracle import bf16 as obf16, estimator, made as omade
    from paper_2106_13308_amd import binding as Bd, inputs

    p = inputs.made_init(n, h, 5)
    p["degrees"] = _degrees(kind, n, h)
    M1, M2 = omade.masks(n, p["degrees"])
    p["W1"], p["W2"] = p["W1"] * M1, p["W2"] * M2
    S = inputs.random_spins(B, n, 6)
    coef = (np.random.default_rng(7).standard_normal(B) / B).astype(np.float32)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.BF16, band=False)
    Sd = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    Sd[:, :n] = torch.from_numpy(S)
    Sd = Sd.cuda()
    q = dict(p, W1=obf16.round_to_bf16(p["W1"]), W2=obf16.round_to_bf16(p["W2"]))
    ref = omade.logp(q, S)
    assert np.abs(Bd.logprob(m, Sd).cpu().numpy() - ref).max() <= 2e-2 * np.abs(ref).max()
    g = estimator.logp_grad(q, S, coef.astype(np.float64))
    dP, db1, db2 = Bd.logprob_backward(m, Sd, torch.from_numpy(coef).cuda())
    dW1, dW2 = m.unpack(dP)
    for name, got in (("W1", dW1), ("W2", dW2), ("b1", db1), ("b2", db2)):
        r = g[name]
        assert np.abs(got.cpu().numpy() - r).max() <= 3e-2 * np.abs(r).max() + 1e-12, name
