"""Receiver nodes of the strip adjoints: all of a row's nodes in a wave's window
are added at once, 64 listed nodes at a time.

Rows with a node on every column (a window of 64 C columns takes up to C runs),
rows whose nodes end one run and begin the next, single nodes at either end of a
window, every lane width, against the plain path's separate injection launches
(another order of FP32 sums: the library's 1e-4, as against the oracle).  And the
time of a launch with many receivers on a narrow grid against that with few: 1.08
times (289 receivers a shot), 1.4 times when the nodes were walked one by one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api as A
    return A


def problem(nz, nx, nt, S, seed):
    rng = np.random.default_rng(seed)
    h, vmax = 5.0, 2400.0
    src = np.stack([rng.uniform(h, (nx - 2) * h, S), rng.uniform(h, (nz - 2) * h, S)], axis=1)
    rho = (2000.0 * (1 + 0.1 * rng.random((nz, nx)))).astype(np.float32)
    K = (rho * (2000.0 * (1 + 0.1 * rng.random((nz, nx)))) ** 2).astype(np.float32)
    return (nz, nx, h, h, 8, nt, 0.5 * h / vmax, vmax), src, K, rho, \
        rng.standard_normal(nt).astype(np.float32), rng


@pytest.mark.parametrize("two,cols", [(2, 1), (2, 2), (1, 1), (1, 2), (1, 4)])
@pytest.mark.parametrize("layout", ["every column", "on nodes", "window ends"])
def test_rows_of_receivers(api, two, cols, layout):
    nz, nx, nt, S = 45, 331, 21, 3
    g, src, K, rho, f, rng = problem(nz, nx, nt, S, cols)
    h = g[2]
    j = np.arange(nx - 1)
    if layout == "every column":    # two full rows of nodes each
        rec = [np.stack([(j + 0.5) * h, np.full(nx - 1, (i + 0.25) * h)], 1) for i in (2, 3, 30)]
    elif layout == "on nodes":      # one node a receiver, rows of 1 to 330 of them
        rec = [np.stack([j[:n] * h, np.full(n, i * h)], 1)
               for i, n in zip(range(3, 43, 3), (1, 63, 64, 65, 127, 128, 129, 330))]
    else:                           # first and last columns of windows of 52 and 58 lanes
        k = np.array([0, 1, 43, 44, 49, 50, 51, 52, 95, 96, 97, 98, 103, 104, 111, 112, 113, 329])
        rec = [np.stack([k * h, np.full(len(k), i * h)], 1) for i in (0, 1, 20, 44 - 2)]
    rec = np.concatenate(rec)
    rec = np.ascontiguousarray(np.broadcast_to(rec, (S,) + rec.shape))
    adj = rng.standard_normal((S, rec.shape[1], nt)).astype(np.float32)
    plain = api.Plan(api.Grid(*g), src, rec, mode="plain")
    ref = [t.double() for t in plain.adjoint("k-rho", K, rho, f, adj)]
    kw = dict(adj_two_step=2, adj_two_step_lane_cols=cols) if two == 2 else \
        dict(adj_two_step=1, lane_cols=cols)
    p = api.Plan(api.Grid(*g), src, rec, shots_per_group=2, **kw)
    for a, b in zip(p.adjoint("k-rho", K, rho, f, adj), ref):
        assert (a - b).abs().max() <= TOL * b.abs().max()


def test_many_receivers_cost_little(api):
    import torch
    nz, nx, nt, S = 367, 250, 48, 40
    g, src, K, rho, f, rng = problem(nz, nx, nt, S, 9)
    c = 0.8 * 0.5 * (nx - 1) * g[2]
    plans = []
    for R in (4, 289):
        th = 2 * np.pi * np.arange(R) / R
        rec = np.stack([0.5 * (nx - 1) * g[2] + c * np.cos(th),
                        0.5 * (nz - 1) * g[2] + c * np.sin(th)], axis=1)
        plans.append(api.Plan(api.Grid(*g), src, rec, two_step=2))
    ws = torch.empty(max(p.workspace_bytes(api.L.FWI_OP_GRADIENT) for p in plans) + 256,
                     dtype=torch.uint8, device="cuda")   # one buffer: its placement counts too
    us = []
    for p in plans:
        adj = torch.ones((S, p.nrec, nt), device="cuda")
        times = []
        for _ in range(4):
            p.forward_keep("k-rho", K, rho, f, ws)
            p.timing(True)
            p.adjoint_kept("k-rho", K, rho, f, adj, ws)
            n, ms = p.timing_read()["adj_pair"]
            p.timing(False)
            times.append(ms / n)
        us.append(min(times) * 1e3)
    assert us[1] <= 1.2 * us[0], us
