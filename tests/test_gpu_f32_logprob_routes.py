"""log pi in FP32 on either side of each line between its two engines, within the FP32 bar of the parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

# sites, units and the samples from which the staged engine takes the call
LINES = [(9, 100, 5760), (16, 320, 5760), (128, 128, 8192), (33, 500, 8192), (192, 256, 8192), (192, 31, 12800),
         (500, 192, 30720), (320, 320, 30720)]


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,line", LINES)
def test_either_side(n, h, line):
    from gpu_util import logit_scale, logp_bound
    from oracle import made
    from paper_2106_13308_amd import binding as Bd
    from paper_2106_13308_amd import inputs

    p = inputs.made_init(n, h, 5)
    M1, M2 = made.masks(n, p["degrees"])
    p["W1"], p["W2"] = p["W1"] * M1, p["W2"] * M2
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.F32, band=False)
    s = inputs.random_spins(line + 1, n, 6)
    S = torch.zeros(line + 1, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(s)
    S = S.cuda()
    for B in (line - 1, line, line + 1):
        rows = np.unique(np.r_[0:70, B // 2:B // 2 + 70, B - 70:B])
        f, sc = logit_scale(p, s[rows])
        lp, Z = Bd.logprob(m, S[:B], want_z=True)
        assert (np.abs(Z.cpu().numpy()[rows, :n] - f["Z"]) <= 1e-5 * sc["z"] + 1e-30).all(), B
        assert (np.abs(lp.cpu().numpy()[rows] - f["logp"]) <= logp_bound(f, s[rows], sc["z"], 1e-5)).all(), B
