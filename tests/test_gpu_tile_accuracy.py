"""Tile kernels over many steps: their adjoint wavefields round as the strip
kernels' do, so that the gradients of a model that is homogeneous but for an
anomaly (every node rounds its coefficients the same way, and a difference in
them adds up along a wave's path) agree after long runs.

The wavefields being the same bit for bit, the gradients differ by the rounding
of their running sums alone: half an ulp, 2^-24, at each of the 40 to 60
launches during which a pulse of about 100 steps passes a node, which add up
like a random walk, 2^-24 sqrt(45) = 4e-7 of the gradient.  Measured 1.4 to
2.2e-7; 5.9 to 7.2e-7 with 1 / h multiplied into the adjoint's coefficients,
which then are another rounded medium than the forward sweep's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BOUND = 2.0 ** -24 * 45 ** 0.5


@pytest.mark.parametrize("n,nt,vmax", [(401, 1600, 2100.0), (801, 2400, 2400.0)])
@pytest.mark.parametrize("ckpt", [0, 32])
def test_long_runs_agree_with_strips(n, nt, vmax, ckpt):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api
    h, fpeak = 5.0, 25.0
    dt = 0.5 * h / vmax
    c = 0.5 * (n - 1) * h
    th = 2.0 * np.pi * np.arange(60) / 60
    rec = np.stack([c + 0.8 * c * np.cos(th), c + 0.8 * c * np.sin(th)], axis=1)
    src = np.array([[c + 0.8 * c * np.cos(0.94), c + 0.8 * c * np.sin(0.94)]])
    z, x = np.mgrid[0:n, 0:n] - 0.5 * n
    bump = 0.1 * np.exp(-(z * z + x * x) / 20.0)
    rho = 2000.0 * (1.0 + bump)
    K = (rho * (2000.0 * (1.0 + bump)) ** 2).astype(np.float32)
    a = (np.pi * fpeak * (np.arange(nt) * dt - 1.5 / fpeak)) ** 2
    f = ((1.0 - 2.0 * a) * np.exp(-a)).astype(np.float32)
    grid = api.Grid(n, n, h, h, 20, nt, dt, vmax)
    out = []
    for kw in ({}, {"two_step": 2}):
        plan = api.Plan(grid, src, rec, ckpt_every=ckpt, **kw)
        d = plan.forward("k-rho", K, rho, f)
        out.append([t.double() for t in (d, *plan.adjoint("k-rho", K, rho, f, d))])
    assert torch.equal(out[0][0], out[1][0])
    for t, s in zip(out[0][1:], out[1][1:]):
        assert (t - s).norm() <= BOUND * s.norm()
