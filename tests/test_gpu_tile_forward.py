"""Plans between the sizes of the two tile rules, where a forward call runs on
the tile kernels and a gradient on the strip kernels: both give what a plan of
strip kernels gives, bit for bit, in either order of the calls, with an odd
number of shots (the strip kernels' groups are padded) and more levels than
are sampled at a time."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,nx,npml,nt,S", [(560, 559, 20, 17, 7), (201, 401, 40, 70, 19)])
def test_forward_on_tiles_gradient_on_strips(nz, nx, npml, nt, S):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api
    rng = np.random.default_rng(nz + S)
    h, vmax = 5.0, 2400.0
    rec = np.stack([rng.uniform(0, (nx - 1.01) * h, 23), rng.uniform(0, (nz - 1.01) * h, 23)],
                   axis=1)
    src = np.stack([rng.uniform(h, (nx - 2) * h, S), rng.uniform(h, (nz - 2) * h, S)], axis=1)
    grid = api.Grid(nz, nx, h, h, npml, nt, 0.5 * h / vmax, vmax)
    vp = (2000.0 * (1 + 0.1 * rng.random((nz, nx)))).astype(np.float32)
    rho = (2000.0 * (1 + 0.1 * rng.random((nz, nx)))).astype(np.float32)
    f = rng.standard_normal(nt).astype(np.float32)
    obs = rng.standard_normal((S, 23, nt)).astype(np.float32)
    default, strips = api.Plan(grid, src, rec), api.Plan(grid, src, rec, two_step=2)
    want = strips.forward("vp-rho", vp, rho, f)
    grads = strips.gradient("vp-rho", vp, rho, f, obs)
    for _ in range(2):
        assert torch.equal(default.forward("vp-rho", vp, rho, f), want)
        for a, b in zip(default.gradient("vp-rho", vp, rho, f, obs), grads):
            assert torch.equal(a, b)
