"""The BF16 hidden adjoint on the masked copy of P^T (sampler tables given) against the one that masks P^T itself."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one entry; ragged tiles and stages; few units that feed many sites each; the 128 x 128 tiles; staircases that jump
SHAPES = [(2, 1, 1, "default"), (65, 63, 65, "default"), (97, 33, 31, "default"), (3000, 30, 70, "default"),
          (70, 2000, 4097, "default"), (300, 300, 100, "first"), (300, 300, 100, "last"), (1300, 700, 66, "clustered")]


@pytest.mark.parametrize("n,h,B,kind", SHAPES)
def test_masked_copy(n, h, B, kind):
    """The same products in the same order, zeros besides: the same bits, in the gradient and in the SR Gram."""
    from paper_2106_13308_amd import binding as Bd, inputs

    p = inputs.made_init(n, h, 5)
    deg = {"default": p["degrees"], "first": np.ones(h, np.int32), "last": np.full(h, n - 1, np.int32),
           "clustered": np.sort(np.random.default_rng(4).choice([1, n // 3, n - 2], size=h)).astype(np.int32)}[kind]
    m = Bd.Made.from_dense(p["W1"], p["b1"], p["W2"], p["b2"], deg, wdtype=Bd.BF16)
    S, _, Zs, Rt = Bd.sample_fwd(m, B, 3, 1)
    coef = torch.randn(B, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")

    def run():
        return (*Bd.backward_sampled(m, S, coef, Zs, Rt), Bd.sr_gram_sampled(m, S, Zs, Rt))

    got = run()
    m.band = None
    for a, b in zip(got, run()):
        assert torch.equal(a, b)
