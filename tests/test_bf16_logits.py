"""The logits behind log pi in BF16, one by one, at the edges of the products' tiles, stages and staircases, within the
BF16 bar of the parity tests: 2e-2 of the sum of a logit's summands' sizes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

# sites, units, samples, degrees: one entry; one more or less than a 64-tile and a 64-column stage; odd and even numbers
# of 32-unit steps; up to 64 sites and units (the staged kernels) and just past; site tiles that are no multiple of eight
SHAPES = [(2, 1, 1, "default"), (64, 64, 64, "default"), (65, 63, 65, "default"), (97, 33, 31, "default"),
          (129, 257, 190, "default"), (40, 900, 70, "default"), (900, 40, 130, "default"), (300, 300, 100, "first"),
          (300, 300, 100, "last"), (1300, 700, 66, "clustered"), (70, 2049, 1030, "default"), (1100, 1030, 70, "default"),
          (128, 200, 16390, "default")]


def _model(n, h, B, kind):
    from gpu_util import logit_scale
    from oracle import bf16, made
    from paper_2106_13308_amd import inputs

    p = inputs.made_init(n, h, 5)
    p["degrees"] = {"default": p["degrees"], "first": np.ones(h, np.int32), "last": np.full(h, n - 1, np.int32),
                    "clustered": np.sort(np.random.default_rng(4).choice([1, n // 3, n - 2], size=h)).astype(np.int32)}[kind]
    M1, M2 = made.masks(n, p["degrees"])
    p["W1"], p["W2"] = p["W1"] * M1, p["W2"] * M2
    s = inputs.random_spins(B, n, 6)
    q = dict(p, W1=bf16.round_to_bf16(p["W1"]), W2=bf16.round_to_bf16(p["W2"]))
    f, sc = logit_scale(q, s)
    return p, q, s, f, sc["z"], 2e-2 * sc["z"] + 1e-30


@pytest.mark.parametrize("n,h,B,kind", [x for x in SHAPES if x[1] > 32])
def test_bar_sees_a_lost_step(n, h, B, kind):
    """A product that drops 32 units, the first or the last of those that feed a site, is past the bar."""
    from oracle import made

    B = min(B, 200)
    p, q, s, f, _, bar = _model(n, h, B, kind)
    for k in (slice(0, 32), slice(h - 32, h)):
        W2 = np.array(q["W2"])
        W2[:, k] = 0
        assert (np.abs(made.forward(dict(q, W2=W2), s)["Z"] - f["Z"]) > bar).any()


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,B,kind", SHAPES)
def test_logits(n, h, B, kind):
    from gpu_util import logp_bound
    from paper_2106_13308_amd import binding as Bd

    p, q, s, f, zscale, bar = _model(n, h, B, kind)
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], p["degrees"], wdtype=Bd.BF16, band=False)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(s)
    lp, Z = Bd.logprob(m, S.cuda(), want_z=True)
    assert (np.abs(Z[:, :n].cpu().numpy() - f["Z"]) <= bar).all()
    assert (np.abs(lp.cpu().numpy() - f["logp"]) <= logp_bound(f, s, zscale, 2e-2)).all()
