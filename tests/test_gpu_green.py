"""Green tables against scipy's FP64 Hankel functions, entry by entry, across
the branches of the evaluation (k r = 8, the quadrants of the argument
reduction, very small and large k r), with table shapes around the pieces of 256
entries and the runs of 64 frequencies.

Tolerance: an entry is an FP64 value rounded to FP32 in each component, half an
ulp = 2^-24 of the component; the FP64 value is good to 4e-13 of |H| from the
fits, and at k r <= 1e4 to another 1e4 x 2^-52 = 2e-12 from the rounding of k r."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EDGES = [1e-6, 1e-3, 0.5, 0.89357697, 2.0, 7.9999995, 8.0, 8.000001, 12.0, 100.53096, 1e4]


@pytest.mark.parametrize("F,C,P", [(1, 11, 1), (3, 40, 257), (65, 13, 7), (130, 1, 1),
                                   (2, 300, 31)])
def test_green_entries(F, C, P):
    torch = pytest.importorskip("torch")
    special = pytest.importorskip("scipy.special")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import born
    rng = np.random.default_rng(F + C + P)
    omega = np.geomspace(1.0, 60.0, F).astype(np.float32)
    cells = np.zeros((C, 2), np.float32)
    cells[:, 0] = (EDGES + list(rng.uniform(0.01, 160.0, max(0, C - 11))))[:C]
    pts = np.zeros((P, 2), np.float32)
    pts[1:, :] = rng.uniform(-3.0, 3.0, (P - 1, 2))
    if C > 12 and P > 2:
        pts[2] = cells[12]
    out = born.green(*(torch.as_tensor(t, device="cuda") for t in (omega, cells, pts)), 4.0, 16.0)
    k = omega.astype(np.float64) * 2.0
    d = cells.astype(np.float64)[:, None] - pts.astype(np.float64)[None]
    r = np.hypot(d[..., 0], d[..., 1])[None]
    self_cell = np.broadcast_to(r == 0, (F, C, P))
    z = k[:, None, None] * np.where(r > 0, r, 1.0)
    keep = ~self_cell & (z <= 1e4)
    h1 = -4j * k[:, None, None] * special.hankel1(1, z) / np.where(r > 0, r, 1.0)
    for g, ref in zip(out, (4j * special.hankel1(0, z), h1 * d[None, ..., 0],
                            h1 * d[None, ..., 1])):
        g = g.cpu().numpy()
        assert np.all(g[self_cell] == 0)
        g, ref = g[keep].astype(np.complex128), ref[keep]
        for part, want in ((g.real, ref.real), (g.imag, ref.imag)):
            bound = 2.0 ** -24 * np.abs(want) + 1e-11 * np.abs(ref) + 1e-44
            assert np.all(np.abs(part - want) <= bound)
