"""Receiver nodes beyond what the strip kernels' packed lists hold: more than 2^23
of them in one strip (two receivers a cell side over 162000 rows of 52 nodes).  The
adjoint then takes one-step launches with R^T r and its imaging term added by
launches of their own, and the forward kernel stores whole intermediate levels.
Against the plain path, within FP32 rounding (the library's 1e-4)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-4


def test_more_nodes_than_a_list_holds():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api
    nz, nx, nt, S, h, vmax = 162000, 52, 5, 2, 5.0, 2400.0
    rng = np.random.default_rng(1)
    # centres of every other cell: four nodes each, every node of the grid once
    x, z = np.meshgrid((2 * np.arange(nx // 2) + 0.5) * h, (2 * np.arange(nz // 2) + 0.5) * h)
    rec = np.stack([x.ravel(), z.ravel()], axis=1)
    assert 4 * len(rec) == nz * nx and (nz - 1) * nx >= 1 << 23
    src = np.array([[100.0, 3e5], [130.0, 8.09e5]])
    grid = api.Grid(nz, nx, h, h, 0, nt, 0.5 * h / vmax, vmax)
    g = torch.Generator(device="cuda").manual_seed(3)
    rho = 2000.0 + 200.0 * torch.rand((nz, nx), generator=g, device="cuda")
    K = rho * (2000.0 + 200.0 * torch.rand((nz, nx), generator=g, device="cuda")) ** 2
    f = torch.as_tensor(rng.standard_normal(nt).astype(np.float32), device="cuda")
    out = []
    for kw in ({"mode": "plain"}, {"shots_per_group": 2}):
        p = api.Plan(grid, src, rec, **kw)
        if "mode" not in kw:
            assert p.info["adj_two_step"] == 0 and p.info["two_step"] == 1
        d = p.forward("k-rho", K, rho, f)
        adj = torch.randn(d.shape, generator=torch.Generator(device="cuda").manual_seed(4),
                          device="cuda")
        p.timing(True)
        out.append((d, *p.adjoint("k-rho", K, rho, f, adj)))
        if "mode" not in kw:
            n = p.timing_read()
            assert n["adj_step"][0] == nt and n["adj_pair"][0] == 0
            assert n["inject"][0] >= nt        # one a step (both shots), and the staging
    for a, b in zip(out[1], out[0]):
        assert (a - b).abs().max() <= TOL * b.abs().max()


@pytest.mark.parametrize("n,nt,ckpt", [(1340, 75, 0), (2100, 33, 0), (2100, 33, 9)])
def test_dense_receivers_stage_fewer_steps(n, nt, ckpt):
    """A receiver on every node: R^T r is staged in at most 256 MB (36 and 12 steps
    at a time, on tiles and on strips), against the plain path; and the gradient's
    workspace does not grow with 64 steps of every node."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api
    h, vmax = 5.0, 2400.0
    rng = np.random.default_rng(n)
    x, z = np.meshgrid((2 * np.arange(n // 2) + 0.5) * h, (2 * np.arange(n // 2) + 0.5) * h)
    rec = np.stack([x.ravel(), z.ravel()], axis=1)
    grid = api.Grid(n, n, h, h, 0, nt, 0.5 * h / vmax, vmax)
    src = [[0.4 * n * h, 0.55 * n * h]]
    gen = torch.Generator(device="cuda").manual_seed(n)
    rho = 2000.0 + 200.0 * torch.rand((n, n), generator=gen, device="cuda")
    K = rho * (2000.0 + 200.0 * torch.rand((n, n), generator=gen, device="cuda")) ** 2
    f = torch.as_tensor(rng.standard_normal(nt).astype(np.float32), device="cuda")
    adj = torch.randn((1, len(rec), nt), generator=gen, device="cuda")
    plans = [api.Plan(grid, src, rec, mode="plain", ckpt_every=ckpt),
             api.Plan(grid, src, rec, ckpt_every=ckpt)]
    got = [p.adjoint("k-rho", K, rho, f, adj) for p in plans]
    for a, b in zip(got[1], got[0]):
        assert (a - b).abs().max() <= TOL * b.abs().max()
    few = api.Plan(grid, src, rec[:1], ckpt_every=ckpt)
    op = api.L.FWI_OP_GRADIENT
    # traces and residuals, the plan's tables (48 bytes a node at most in all of
    # them), and what is staged
    more = 2 * 4 * len(rec) * nt + 80 * n * n + (256 << 20) + (8 << 20)
    assert plans[1].workspace_bytes(op) - few.workspace_bytes(op) <= more
