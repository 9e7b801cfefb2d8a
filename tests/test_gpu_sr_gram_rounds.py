"""The BF16 SR Gram where the tiles just pass a full round of workgroups (513 to 576 tiles of 64 x 64 samples): the rest
runs as quadrants of one wave each.  Oracle and error bar of test_gpu_sr.py (derived there)."""
import numpy as np
import pytest
import torch

from paper_2106_13308_amd import inputs

from gpu_util import DEV, build_made, oracle_params
from test_gpu_sr import check_gram

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,B", [(67, 70, 2048), (40, 33, 1990), (9, 2, 2050)])
def test_sr_gram_short_last_round(n, h, B):
    from paper_2106_13308_amd import binding as Bd
    print(f"[sr-gram] rounds n={n} h={h} B={B}", flush=True)
    p = inputs.made_init(n, h, 91)
    S = inputs.random_spins(B, n, 92)
    Sd = torch.zeros((B, Bd.ld(n)), dtype=torch.int8, device=DEV)
    Sd[:, :n] = torch.from_numpy(S).to(DEV)
    made = build_made(p, Bd.BF16)
    K = Bd.sr_gram(made, Sd, B)
    torch.cuda.synchronize()
    K = K.double().cpu().numpy()
    assert np.array_equal(K, K.T)
    check_gram(K, oracle_params(p, Bd.BF16), S, "bf16")
