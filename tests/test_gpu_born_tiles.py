"""Born data and gradient at the edges of their matrix-core tiles, against FP64
sums over the very tables the kernels read: receivers below, at and past a
group of 32 (odd ones too, whose last group is moved back) and past a chunk of
16, cells past a chunk of 16 and a block of 64, sources past a tile and a group
of tiles, one source, and more frequencies than one block sums.

Tolerance, relative 2-norm 2e-6: a product of two complex entries is good to
about 4 x 2^-24 (three bf16 parts of 24 bits, six of their nine products, the
coefficient's own rounding), the sums run through at most 18 x 8 dependent FP32
additions of matrix instructions, whose random roundings add up to sqrt(144) x
2^-24 of the running sum; together about 1e-6 with the sum not far below the
terms' root sum of squares."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,S,R,C", [(1, 1, 1, 1), (2, 9, 31, 17), (1, 16, 32, 64),
                                     (3, 17, 33, 65), (2, 48, 63, 15), (1, 65, 129, 100),
                                     (5, 3, 47, 81), (9, 64, 16, 130)])
def test_edges(F, S, R, C):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import born
    rng = np.random.default_rng(1000 * F + S + R + C)
    omega = np.linspace(20.0, 90.0, F).astype(np.float32)
    spec = (rng.normal(size=F) + 1j * rng.normal(size=F)).astype(np.complex64)
    src, rec = rng.uniform(-400, 400, (S, 2)), rng.uniform(-400, 400, (R, 2))
    cells = rng.uniform(-100, 100, (C, 2))
    prob = born.BornProblem(omega, spec, src, rec, cells, 25.0, 8e9, 2000.0)
    xK, xR = (rng.uniform(-0.2, 0.2, C).astype(np.float32) for _ in range(2))
    q = (rng.normal(size=(F, S, R)) + 1j * rng.normal(size=(F, S, R))).astype(np.complex64)
    d = prob.data(xK, xR, direct=False).cpu().numpy()
    gK, gR = (t.cpu().numpy() for t in prob.gradient(torch.as_tensor(q, device="cuda")))
    Gs, Gr = ([t.cpu().numpy().astype(np.complex128) for t in g] for g in (prob.Gs, prob.Gr))
    w2, aK, aR = omega.astype(np.float64)[:, None] ** 2, 25.0 / 8e9, -25.0 / 2000.0
    want = np.einsum("fcs,fcr,fc->fsr", Gs[0], Gr[0], aK * w2 * xK)
    for a, b in zip(Gs[1:], Gr[1:]):
        want += np.einsum("fcs,fcr,c->fsr", a, b, aR * xR)
    want *= spec.astype(np.complex128)[:, None, None]
    W = np.conj(q.astype(np.complex128)) * spec.astype(np.complex128)[:, None, None]
    t = [np.einsum("fsr,fcr,fcs->fc", W, b, a).real for a, b in zip(Gs, Gr)]
    wK, wR = aK * (w2 * t[0]).sum(0), aR * (t[1] + t[2]).sum(0)
    for got, ref in ((d, want), (gK, wK), (gR, wR)):
        assert np.linalg.norm(got - ref) <= 2e-6 * np.linalg.norm(ref)
