"""The sparse energies at the edges of their row shares and byte lanes, against the exact oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (sites, edges or None for all pairs, weights lo..hi, batch): fewer edges than a load takes; rows shorter and
# longer than a lane's share, up to 64 lanes a row; empty rows; weights that fill a byte, pass it
# and are negative; batches that end inside a group of eight; the row pointer outside LDS
SHAPES = [(2, 1, 1, 1, 1), (9, 3, 1, 5, 7), (40, 4, 1, 1, 8), (33, None, 1, 1, 9), (150, None, 0, 255, 16), (300, None, 1, 3, 5),
          (700, None, -4, 300, 11), (2100, None, 1, 1, 3), (5000, 2500, 1, 9, 13), (17000, 60000, 1, 5, 10)]


@pytest.mark.parametrize("n,m,lo,hi,B", SHAPES)
def test_csr_energies(n, m, lo, hi, B):
    """Integer weights exactly; float weights within the rounding of a sum in double precision, 2^-52 per addition
    of terms up to the sum of |w|."""
    from oracle import energy as oen
    from paper_2106_13308_amd import binding as Bd, inputs

    rng = np.random.default_rng(n)
    if m is None:
        edges = np.stack(np.triu_indices(n, 1), 1).astype(np.int32)
    else:
        e = rng.integers(0, n, (8 * m + 8, 2))
        e = np.unique(np.sort(e[e[:, 0] != e[:, 1]], axis=1), axis=0)
        edges = e[rng.permutation(len(e))[:m]].astype(np.int32)
    S = inputs.random_spins(B, n, 2)
    Sd = torch.zeros((B, Bd.ld(n)), dtype=torch.int8, device="cuda")
    Sd[:, :n] = torch.from_numpy(S).cuda()
    w = rng.integers(lo, hi + 1, len(edges)).astype(np.int32)
    got = Bd.energy(Bd.Hamiltonian.from_edges(n, edges, w, device="cuda"), Sd).cpu().numpy()
    assert got.dtype == np.int64 and np.array_equal(got, oen.energy_edges(edges, w, S))
    wf = rng.uniform(-1, 1, len(edges)).astype(np.float32)
    got = Bd.energy(Bd.Hamiltonian.from_edges(n, edges, wf, device="cuda"), Sd).cpu().numpy()
    ref = oen.energy_edges(edges, wf.astype(np.float64), S)
    assert np.abs(got - ref).max() <= 2.0 ** -52 * 64 * np.abs(wf.astype(np.float64)).sum()
