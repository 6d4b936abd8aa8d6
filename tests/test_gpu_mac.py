"""The far sums of 10 to 16 targets: groups of 12, 15 or 18 lags without a test, then guarded ones."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# bars of 11 lags (fewer than a group, and fewer than the 16 targets: the launch for the next block has no lag
# at all) and 40 lags (two or three groups and a remainder)
@pytest.mark.parametrize("tb,ob,ov", [(10, 0, 0), (12, 0, 0), (14, 0, 0), (16, 0, 0), (4, 12, 1), (4, 16, 1),
                                      (4, 12, 2), (4, 16, 2)])
@pytest.mark.parametrize("UVW,ell,nr", [((8, 4, 2), 11, 2), ((38, 3, 2), 40, 1)])
def test_far_sums_against_step_by_step(torch_cuda, UVW, ell, nr, tb, ob, ov):
    """A march with time blocks against one that sums every step's lags at once (64-bit sums in another order,
    and a solve to 1e-13 of it: <= 1e-11), over several turns of the ring; a second march after a reset
    repeats the first bit for bit."""
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    U, V, W = UVW
    n = 2 * ell + 37
    eps = wl.random_eps(U, V, W, 5, 1.5, 9.0)
    waves = [wl.gaussian_wave(U, V, W, k, p, 3.0) for k, p in wl.random_directions(nr, 7)]
    prob = wl.Problem("bar", U, V, W, eps, waves, n, fir=wl.binomial_highpass(3, 0.01))
    out = []
    for cfg in (dict(time_block=1), dict(time_block=tb, outer_block=ob, outer_overlap=ov)):
        s = motjvie.solver_for(prob, cg_rtol=1e-13, **cfg)
        assert s.ell == ell
        assert cfg["time_block"] == 1 or s.info()["outer_block"] == ob
        for _ in range(2):
            J = torch.zeros((n, nr, 3, W, V, U), dtype=torch.float64, device="cuda")
            s.run(n, J)
            out.append(J)
            s.reset()
        s.close()
    assert torch.equal(out[0], out[1]) and torch.equal(out[2], out[3])
    a, b = (J.cpu().numpy() for J in out[1:3])
    assert np.isfinite(b).all() and np.abs(a).max() > 0
    assert np.linalg.norm(a - b) <= 1e-11 * np.linalg.norm(a)
