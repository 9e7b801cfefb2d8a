"""The sparse integer energies for weights that do not fit the byte lanes, in both forms of the kernel (four rows at a
time, or two with two workgroups a CU: batches past 2048), against the exact oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# both signs, a byte and more, 16 bits and more, next to weights that do fit
WEIGHTS = [(-1, 1), (2046, -2047), (16, 15), (40, 1), (255, 0), (256, 1), (32767, -32768), (-1, 70000), (2**31 - 1, -2**31)]


@pytest.mark.parametrize("n,B", [(130, 9), (150, 2051), (2300, 2049)])
@pytest.mark.parametrize("w", WEIGHTS)
def test_csr_weights(n, B, w):
    """All pairs (n = 2300: a path with chords), weights of the two values at random or the first alone; strings at random,
    alternating (half of all pairs of unequal spins) and all equal."""
    from oracle import energy as oen
    from paper_2106_13308_amd import binding as Bd, inputs

    rng = np.random.default_rng(n)
    edges = np.stack(np.triu_indices(n, 1), 1) if n < 2000 else np.concatenate(
        [np.stack([np.arange(n - k), np.arange(k, n)], 1) for k in (1, 2, 7, 30, 900)])
    edges = edges.astype(np.int32)
    picks = sorted({0, 1, 2, B // 2, B - 1})
    S = torch.zeros(B, Bd.ld(n), dtype=torch.int8)
    S[:, :n] = torch.from_numpy(inputs.random_spins(B, n, 2))
    S[0, :n] = torch.from_numpy((1 - 2 * (np.arange(n) % 2)).astype(np.int8))
    S[1, :n] = 1
    Sd = S.cuda()
    for wt in (rng.choice(w, len(edges)), np.full(len(edges), w[0])):
        wt = wt.astype(np.int32)
        E = Bd.energy(Bd.Hamiltonian.from_edges(n, edges, wt), Sd).cpu().numpy()
        assert np.array_equal(E[picks], oen.energy_edges(edges, wt, S[picks, :n].numpy()))
