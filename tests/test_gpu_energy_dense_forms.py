"""Every form of the dense energy's kernels, on both sides of the rules that choose between them, and rows whose
entries lie too far apart for a common fixed point."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# all rows in FP64 up to 160 sites; then 2, 4 (16 rows) or 8 waves (32 rows) a workgroup, J by 16 bytes (n a multiple
# of four) or by single entries, batches and sites that end inside a tile
SHAPES = [(160, 70), (161, 33), (164, 129), (1003, 1000), (2000, 1003), (2001, 1003), (2000, 8161), (2001, 8161)]


def _batch(n, B):
    from paper_2106_13308_amd import binding as Bd

    g = torch.Generator(device="cuda").manual_seed(n + B)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8, device="cuda")
    S[:, :n] = 2 * torch.randint(0, 2, (B, n), generator=g, device="cuda", dtype=torch.int8) - 1
    return S


def _energy(J, S):
    from paper_2106_13308_amd import binding as Bd

    return Bd.energy(Bd.Hamiltonian.dense(J + J.T), S).cpu().numpy()


def _picks(B):
    return sorted({0, 1, B // 2, B - 2, B - 1})


def _exact(J, s):
    i, j = np.nonzero(J)
    return math.fsum(J[i, j].astype(np.float64) * (s[i].astype(np.float64) * s[j]))


@pytest.mark.parametrize("n,B", SHAPES)
def test_dense_forms(n, B):
    """Against exact sums.  A row's sum is rounded to double a few times (2^-53 of at most sum |J_i.|), and so are the
    sums over the rows: 2^-50 of sum |J| in all."""
    J = np.triu(np.random.default_rng(n).standard_normal((n, n)), 1).astype(np.float32)
    S = _batch(n, B)
    E = _energy(J, S)
    for b in _picks(B):
        ref = _exact(J, S[b, :n].cpu().numpy())
        assert abs(E[b] - ref) <= 2.0 ** -50 * np.abs(J.astype(np.float64)).sum(), b


@pytest.mark.parametrize("n,B", SHAPES)
def test_dense_cancelling_penalties(n, B):
    """Rows that begin with two penalties of opposite sign on equal spins, 2^45 against couplings in steps of 2^-20:
    summed in double in the order of the columns every partial sum is exact, so the energy is exact."""
    rng = np.random.default_rng(n)
    J = np.triu(rng.integers(-1000, 1001, (n, n)), 1).astype(np.float32) * np.float32(2.0 ** -20)
    S = _batch(n, B)
    for i in (0, 19, 70, n - 8):
        c = (i + 4) // 4 * 4  # an aligned group of four columns
        J[i, :c + 4] = 0.0
        J[i, c], J[i, c + 1] = 2.0 ** 45, -2.0 ** 45
        S[:, c + 1] = S[:, c]
    E = _energy(J, S)
    for b in _picks(B):
        assert E[b] == _exact(J, S[b, :n].cpu().numpy()), b


@pytest.mark.parametrize("n,B", [(2000, 1003), (2001, 8161)])
def test_dense_forms_non_finite(n, B):
    J = np.triu(np.random.default_rng(n).standard_normal((n, n)), 1).astype(np.float32)
    J[70, 1500] = np.inf
    S = _batch(n, B)
    s = (S[:, 70].double() * S[:, 1500].double()).cpu().numpy()
    assert np.array_equal(_energy(J, S), np.where(s > 0, np.inf, -np.inf))
    J[33, 34] = np.nan
    assert np.isnan(_energy(J, S)).all()
