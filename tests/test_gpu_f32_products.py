"""The FP32 products at the edges of their tiles, runs and searches, against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one entry each; ragged 32-tiles; many units per site; many sites per unit; a three-level search of c;
# the 64 x 64 shape in the layers (tiles of ld(B) x ld(h) >= 512) and in the weight gradient
SHAPES = [(2, 1, 1), (33, 31, 33), (65, 100, 31), (64, 64, 64), (20, 700, 70), (1000, 5, 130), (4200, 40, 40),
          (100, 520, 3700), (2100, 1000, 40)]


@pytest.mark.parametrize("n,h,B", SHAPES)
def test_f32_products(n, h, B):
    """log pi within 1e-5 of its size and the gradient of sum_b coef_b log pi within 1e-4 of each
    array's largest entry (the FP32 bars of the parity tests)."""
    from oracle import estimator, made as omade
    from paper_2106_13308_amd import binding as Bd, inputs

    p = inputs.made_init(n, h, 5)
    S = inputs.random_spins(B, n, 6)
    coef = (np.random.default_rng(7).standard_normal(B) / B).astype(np.float32)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.F32, band=False)
    Sd = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    Sd[:, :n] = torch.from_numpy(S)
    Sd = Sd.cuda()
    ref = omade.logp(p, S)
    assert np.abs(Bd.logprob(m, Sd).cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
    g = estimator.logp_grad(p, S, coef.astype(np.float64))
    dP, db1, db2 = Bd.logprob_backward(m, Sd, torch.from_numpy(coef).cuda())
    dW1, dW2 = m.unpack(dP)
    for name, got in (("W1", dW1), ("W2", dW2), ("b1", db1), ("b2", db2)):
        r = g[name]
        assert np.abs(got.cpu().numpy() - r).max() <= 1e-4 * np.abs(r).max() + 1e-12, name
