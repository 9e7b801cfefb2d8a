"""Float couplings on either side of each rule of the row kernel: one lane or several a row, one or two workgroups a CU,
the row pointer in LDS or not."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")


@pytest.mark.gpu
@pytest.mark.parametrize("B", [1, 2048, 2049])
@pytest.mark.parametrize("n,mean", [(767, 20), (768, 20), (768, 31), (768, 32), (2000, 17), (13500, 20), (13500, 40)])
def test_float_rows(n, mean, B):
    """A row's sum is a chain of at most some 60 additions, the sum over rows and lanes one of 40: 2^-46 of sum |w|."""
    from paper_2106_13308_amd import binding as Bd, inputs

    k = np.arange(1, mean + 1)  # a ring with chords: mean edges a row, n * mean in all
    edges = np.sort(np.stack([np.repeat(np.arange(n), mean), (np.repeat(np.arange(n), mean) + np.tile(k * k % (n // 2 - 1) + 1, n)) % n], 1), axis=1)
    edges = np.unique(edges, axis=0).astype(np.int32)
    w = np.random.default_rng(n).standard_normal(len(edges)).astype(np.float32)
    s = inputs.random_spins(B, n, 3)
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(s)
    E = Bd.energy(Bd.Hamiltonian.from_edges(n, edges, w), S.cuda()).cpu().numpy()
    for b in sorted({0, B // 2, B - 1}):
        v = s[b].astype(np.float64)
        ref = math.fsum(w.astype(np.float64) * v[edges[:, 0]] * v[edges[:, 1]])
        assert abs(E[b] - ref) <= 2.0 ** -46 * np.abs(w.astype(np.float64)).sum(), b
