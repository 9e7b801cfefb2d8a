"""vqmc_sr_solve on several streams at once: its back substitution waits between workgroups, which must not depend on
how the workgroups of different solves share the GPU."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [200, 12000])  # few workgroups; together more than the GPU holds at a time
def test_sr_solve_concurrent_streams(B):
    """The arithmetic of a solve does not depend on its schedule: the same bits as one after the other."""
    from paper_2106_13308_amd import binding as Bd

    g = torch.Generator(device="cuda").manual_seed(B)
    jobs = []
    for _ in range(4):
        O = torch.randn(B, 32, generator=g, device="cuda")
        rhs = torch.randn(B, generator=g, device="cuda")
        K = O @ O.T
        K = torch.tril(K) + torch.tril(K, -1).T
        ws = torch.empty(int(Bd.lib.vqmc_sr_solve_workspace_bytes(B)), dtype=torch.uint8, device="cuda")
        jobs.append((K.contiguous(), rhs, ws))
    ref = [Bd.sr_solve(K, 0.5, rhs, 1.0, ws=ws) for K, rhs, ws in jobs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in jobs]
    out = []
    for s, (K, rhs, ws) in zip(streams, jobs):
        with torch.cuda.stream(s):
            out.append(Bd.sr_solve(K, 0.5, rhs, 1.0, ws=ws))
    torch.cuda.synchronize()
    for y, r in zip(out, ref):
        assert torch.isfinite(r).all() and torch.equal(y, r)
