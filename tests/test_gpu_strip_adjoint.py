"""Strip adjoint: odd step counts and segments of odd and even length (a pair
reaches over a segment's start, the last one past the first step), shot groups
with padding shots, receivers on every column of a row (runs of 64 nodes end
inside a row), against one-step launches (bit for bit) and the FP64 oracle, at
a fixed adjoint source."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api as A
    return A


def maxrel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


def problem(nz, nx, npml, nt, S, dense):
    rng = np.random.default_rng(nz + nt + S)
    h, vmax = 5.0, 2400.0
    dt = 0.5 * h / vmax
    src = np.stack([rng.uniform(h, (nx - 2) * h, S), rng.uniform(h, (nz - 2) * h, S)], axis=1)
    if dense:
        j = np.arange(nx - 1)
        rec = np.concatenate([np.stack([(j + 0.5) * h, np.full(nx - 1, (i + 0.25) * h)], axis=1)
                              for i in (2, nz // 2, nz - 3)])
    else:
        rec = np.stack([rng.uniform(0, (nx - 1.01) * h, 23), rng.uniform(0, (nz - 1.01) * h, 23)],
                       axis=1)
    rec = np.ascontiguousarray(np.broadcast_to(rec, (S,) + rec.shape))
    rho = 2000.0 * (1 + 0.1 * rng.random((nz, nx)))
    K = rho * (2000.0 * (1 + 0.1 * rng.random((nz, nx)))) ** 2
    f = rng.standard_normal(nt)
    adj = rng.standard_normal((S, rec.shape[1], nt)).astype(np.float32)
    g = (nz, nx, h, h, npml, nt, dt, vmax)
    ref = O.adjoint_krho(O.Grid(*g), src, rec, K, rho, f, adj.astype(np.float64))
    return g, src, rec, K, rho, f, adj, ref


@pytest.mark.parametrize("spg", [1, 2, 4])
@pytest.mark.parametrize("nt,ckpt,dense", [(1, 0, False), (41, 0, True), (41, 7, False),
                                           (40, 9, True), (70, 8, False)])
def test_pairs_over_segments(api, spg, nt, ckpt, dense):
    g, src, rec, K, rho, f, adj, (eK, er) = problem(61, 150, 8, nt, 3, dense)
    out = []
    for two in (1, 2):
        p = api.Plan(api.Grid(*g), src, rec, shots_per_group=spg, adj_two_step=two,
                     adj_two_step_band_rows=two and 19, ckpt_every=ckpt)
        assert p.info["adj_two_step"] == two - 1
        out.append([t.cpu().numpy() for t in p.adjoint("k-rho", K, rho, f, adj)])
        assert maxrel(out[-1][0], eK) <= TOL and maxrel(out[-1][1], er) <= TOL
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_default_groups_with_padding(api):
    """A problem too large for the tiles, with shots that fill no group."""
    g, src, rec, K, rho, f, adj, (eK, er) = problem(601, 601, 40, 9, 11, False)
    p = api.Plan(api.Grid(*g), src, rec)
    gK, gr = (t.cpu().numpy() for t in p.adjoint("k-rho", K, rho, f, adj))
    assert maxrel(gK, eK) <= TOL and maxrel(gr, er) <= TOL
