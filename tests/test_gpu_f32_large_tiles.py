"""The FP32 products' 64 x 64 tiles in the second layer (512 tiles and more), ragged in sites, units and samples."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the last: an unpadded batch that ends in the first half of a tile's rows, units one past a run of sixteen ks
SHAPES = [(500, 97, 4085), (2085, 49, 1001), (2000, 49, 1044)]


@pytest.mark.parametrize("n,h,B", SHAPES)
def test_f32_large_tiles(n, h, B):
    """The FP32 bars of the parity tests: logits within 1e-5 of the sum of their summands' sizes, log pi within what that
    gives, the gradient of sum_b coef_b log pi within 1e-4 of each array's largest entry."""
    from gpu_util import instance, logit_scale, logp_bound
    from oracle import estimator
    from paper_2106_13308_amd import binding as Bd, inputs

    assert -(-B // 64) * -(-n // 64) >= 512
    p, _ = instance(n, h, seed=5, graph=None, scale=2.0)
    s = inputs.random_spins(B, n, 6)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.F32, band=False)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(s)
    S = S.cuda()
    lp, Z = Bd.logprob(m, S, want_z=True)
    f, sc = logit_scale(p, s)
    assert (np.abs(Z[:, :n].cpu().numpy() - f["Z"]) <= 1e-5 * sc["z"] + 1e-30).all()
    assert (np.abs(lp.cpu().numpy() - f["logp"]) <= logp_bound(f, s, sc["z"], 1e-5)).all()
    coef = (np.random.default_rng(7).standard_normal(B) / B).astype(np.float32)
    g = estimator.logp_grad(p, s, coef.astype(np.float64))
    dP, db1, db2 = Bd.logprob_backward(m, S, torch.from_numpy(coef).cuda())
    dW1, dW2 = m.unpack(dP)
    for name, got in (("W1", dW1), ("W2", dW2), ("b1", db1), ("b2", db2)):
        assert np.abs(got.cpu().numpy() - g[name]).max() <= 1e-4 * np.abs(g[name]).max() + 1e-12, name
