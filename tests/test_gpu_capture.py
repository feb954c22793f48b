"""Gradients, forward calls and Born gradients in a HIP graph: replays on inputs
changed in place give what eager calls give, bit for bit, with eager work and
synchronizations between them.  On the tile kernels, and on the strip kernels with
the whole history and with checkpoints."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def check(torch, change, call):
    """call(): enqueues the work and returns its output tensors (the same ones)."""
    outs = call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        change()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in outs]
        for t in outs:
            t.zero_()
        call()
        torch.cuda.synchronize()
        for a, b in zip(got, outs):
            assert torch.equal(a, b)
            assert torch.isfinite(b).all() and b.abs().max() > 0


@pytest.mark.parametrize("kw", [{}, {"ckpt_every": 9}, {"two_step": 2},
                                {"two_step": 2, "ckpt_every": 9}])
def test_wave_calls(torch, kw):
    from paper_1804_01184_amd import api
    n, nt, S, h = 101, 40, 3, 5.0
    rng = np.random.default_rng(1)
    src = np.stack([rng.uniform(h, 400, S), rng.uniform(h, 400, S)], axis=1)
    rec = np.stack([rng.uniform(h, 400, 17), rng.uniform(h, 400, 17)], axis=1)
    plan = api.Plan(api.Grid(n, n, h, h, 12, nt, 0.001, 2800.0), src, rec, **kw)
    vp = torch.full((n, n), 2000.0, device="cuda")
    rho = torch.full((n, n), 2100.0, device="cuda")
    f = torch.as_tensor(rng.standard_normal(nt).astype(np.float32), device="cuda")
    obs = torch.zeros((S, 17, nt), device="cuda")
    out = (torch.empty(1, device="cuda"), torch.empty_like(vp), torch.empty_like(vp))
    traces = torch.empty_like(obs)

    def call():
        plan.gradient("vp-rho", vp, rho, f, obs, out=out)
        plan.forward("vp-rho", vp, rho, f, traces=traces)
        return [*out, traces]

    check(torch, lambda: vp.mul_(1.02), call)


@pytest.mark.parametrize("S", [3, 20])
def test_born_calls(torch, S):
    from paper_1804_01184_amd import born
    rng = np.random.default_rng(S)
    z, x = np.mgrid[0:21, 0:23] * 5.0
    cells = np.stack([x.ravel(), z.ravel()], axis=1)

    def ring(k):
        return np.stack([50 + 200 * np.cos(np.arange(k)), 50 + 200 * np.sin(np.arange(k))], 1)

    prob = born.BornProblem(np.array([30.0, 60.0, 90.0]), np.ones(3, complex), ring(S), ring(37),
                            cells, 25.0, 8e9, 2000.0, "cuda")
    xk = torch.as_tensor(0.1 * rng.random(len(cells)).astype(np.float32), device="cuda")
    xr = torch.as_tensor(0.1 * rng.random(len(cells)).astype(np.float32), device="cuda")
    hold = []

    def call():
        d = prob.data(xk, xr)
        new = [torch.view_as_real(d), *prob.gradient(d)]
        if not hold:
            hold.extend(t.clone() for t in new)
        for a, b in zip(hold, new):
            a.copy_(b)
        return hold

    check(torch, lambda: xk.mul_(1.1), call)
