"""The dense energy's fixed-point planes: tile edges, rows of very different sizes, entries far below a
row's largest, zero rows, non-finite entries."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _energy(J, s):
    from paper_2106_13308_amd import binding as Bd

    S = torch.zeros(s.shape[0], Bd.ld(s.shape[1]), dtype=torch.int8)
    S[:, :s.shape[1]] = torch.from_numpy(s)
    return Bd.energy(Bd.Hamiltonian.dense(J), S.cuda()).cpu().numpy()


@pytest.mark.parametrize("n,B", [(2, 1), (31, 33), (32, 64), (33, 65), (63, 100), (64, 31), (65, 257), (130, 4500), (1001, 300)])
@pytest.mark.parametrize("spread", [0.0, 12.0])
def test_dense_energy_edges(n, B, spread):
    """Against exact sums (math.fsum over the exact products).  Per row: an entry is off by at most
    2^-54 of the row's bound 2^e <= 2 max |J_i.|, and joining the byte sums and the rows rounds to
    double a few times."""
    import math

    rng = np.random.default_rng(n + B)
    J = (rng.standard_normal((n, n)) * np.exp(spread * rng.standard_normal((n, n)))).astype(np.float32)
    J = np.triu(J, 1)
    if n > 40:
        J[7] = 0.0
    s = (2 * rng.integers(0, 2, (B, n)) - 1).astype(np.int8)
    E = _energy(J + J.T, s)
    Jd = J.astype(np.float64)
    bar = np.sum(2.0 ** -53 * np.abs(Jd).max(axis=1) * n) + 2.0 ** -50 * np.abs(Jd).sum()
    for b in range(0, B, max(1, B // 16)):
        ref = math.fsum((Jd * np.outer(s[b], s[b]).astype(np.float64)).ravel())
        assert abs(E[b] - ref) <= bar


def test_dense_energy_non_finite():
    rng = np.random.default_rng(3)
    n, B = 70, 40
    s = (2 * rng.integers(0, 2, (B, n)) - 1).astype(np.int8)
    J = np.triu(rng.standard_normal((n, n)), 1).astype(np.float32)
    J[5, 60] = np.inf
    assert np.array_equal(_energy(J + J.T, s), np.where(s[:, 5] * s[:, 60] > 0, np.inf, -np.inf))
    J[33, 34] = np.nan
    assert np.isnan(_energy(J + J.T, s)).all()
