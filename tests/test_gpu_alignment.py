"""Spins, weights and workspaces that do not start on a 16-byte boundary, against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _shifted(t, nbytes=8):
    """A copy of t that starts nbytes past a 16-byte boundary"""
    k = nbytes // t.element_size()
    flat = torch.empty(t.numel() + k, dtype=t.dtype, device=t.device)
    assert flat.data_ptr() % 16 == 0
    flat[k:] = t.reshape(-1)
    return flat[k:].view(t.shape)


@pytest.mark.parametrize("what", ["spins", "weights"])
@pytest.mark.parametrize("n,h,B", [(130, 97, 70), (20, 40, 33)])
@pytest.mark.parametrize("wd", ["f32", "bf16"])
def test_unaligned_rows(n, h, B, wd, what):
    """The bars of the aligned calls: logits within 1e-5 (FP32) or 2e-2 (BF16) of the sum of their summands' sizes and
    log pi by what that gives, gradients within 2e-5 or 3e-2 of the largest entry; the Gram within twice that of the
    Gram of aligned inputs (each entry a product of two factors so rounded)."""
    from gpu_util import instance, logit_scale, logp_bound, oracle_params
    from oracle import estimator
    from paper_2106_13308_amd import binding as Bd, inputs

    wdtype = Bd.F32 if wd == "f32" else Bd.BF16
    rtol, gtol = (1e-5, 2e-5) if wd == "f32" else (2e-2, 3e-2)
    p, _ = instance(n, h, seed=5, graph=None, scale=2.0)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=wdtype, band=False)
    s = inputs.random_spins(B, n, 7)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(s)
    S = S.cuda()
    K0 = Bd.sr_gram(m, S)
    if what == "spins":
        S = _shifted(S)
    else:
        m.P, m.Pt = _shifted(m.P), _shifted(m.Pt)
    assert (S.data_ptr() | m.P.data_ptr()) % 16 == 8
    q = oracle_params(p, wdtype)
    f, sc = logit_scale(q, s)
    bound = logp_bound(f, s, sc["z"], rtol)
    lp, Z = Bd.logprob(m, S, want_z=True)
    assert (np.abs(Z[:, :n].cpu().numpy() - f["Z"]) <= rtol * sc["z"] + 1e-30).all()
    assert (np.abs(lp.cpu().numpy() - f["logp"]) <= bound).all()
    assert (np.abs(Bd.logprob_noalloc(m, S).cpu().numpy() - f["logp"]) <= bound).all()
    coef = (np.random.default_rng(9).standard_normal(B) / B).astype(np.float32)
    g = estimator.logp_grad(q, s, coef.astype(np.float64))
    dP, db1, db2 = Bd.logprob_backward(m, S, torch.from_numpy(coef).cuda())
    dW1, dW2 = m.unpack(dP)
    for name, got in (("W1", dW1), ("W2", dW2), ("b1", db1), ("b2", db2)):
        assert np.abs(got.cpu().numpy() - g[name]).max() <= gtol * np.abs(g[name]).max() + 1e-12, name
    K = Bd.sr_gram(m, S)
    assert (K - K0).abs().max() <= 2 * gtol * K0.abs().max()


@pytest.mark.parametrize("wd", ["f32", "bf16"])
def test_unaligned_workspace(wd):
    from gpu_util import instance
    from paper_2106_13308_amd import binding as Bd, inputs

    n, h, B = 130, 97, 70
    p, _ = instance(n, h, seed=5, graph=None)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.F32 if wd == "f32" else Bd.BF16, band=False)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(inputs.random_spins(B, n, 7))
    S = S.cuda()
    ws = torch.empty(Bd.workspace(Bd.WS_LOGPROB, m, B).numel() + 8, dtype=torch.uint8, device="cuda")
    ref = Bd.logprob(m, S)
    # the same products in another FP32 order
    assert (Bd.logprob(m, S, ws=ws[8:]) - ref).abs().max() <= (1e-5 if wd == "f32" else 2e-2) * ref.abs().max()
