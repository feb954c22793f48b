"""Shots that only fill up a group of the two-step adjoint never cost a plan its
whole pressure history: with 30 shots of 1081 x 1081 nodes and as many steps as
half of the device memory holds for 30 records a level, the 32 of four shots a
wave would not fit.  (Plans hold host memory only.)"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [30, 46, 54])
def test_padding_keeps_the_whole_history(S):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_01184_amd import api
    n, npml, h = 1001, 40, 5.0
    N = (n + 2 * npml) ** 2
    record = (N + N - n * n + 63) // 64 * 64 + 1024      # floats of a level
    budget = torch.cuda.mem_get_info()[1] // 2
    even = S + S % 2
    nt = int(budget // (even * record * 4)) - 1          # nt + 1 levels
    grid = api.Grid(n, n, h, h, npml, nt, 0.001, 2400.0)
    src = [[500.0 + 50.0 * s, 2000.0] for s in range(S)]
    p = api.Plan(grid, src, [[600.0, 640.0], [800.0, 801.0]])
    assert p.info["ckpt_every"] == nt and p.info["segments"] == 1
