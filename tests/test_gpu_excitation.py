"""Voxel averages of the incident pulse by the Gaussian's series, and the forms beyond it."""
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


def _unit(*v):
    v = np.asarray(v, float)
    return v / np.linalg.norm(v)


# pulse (standard deviation in voxels) and direction of each wave.  "series": all of them take it, from 5 terms
# to 16, and an axis wave whose spread needs more than an 8-point rule's; "mixed": erf on the widest axis
# and an axis wave beyond the series beside two that take it, in the build for every form
CASES = {"series": [(8.0, (-1, -1, -2 ** 0.5)), (1.2, (1, 1, 1)), (1.01, (1, -1, 1)), (0.6, (0, 0, 1))],
         "mixed": [(0.45, (0.94, 0.32, 0.1)), (0.35, (0, 1, 0)), (3.0, (0.3, 0.5, -0.8)), (2.0, (1, 0, 0))]}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("prism", [False, True])
def test_series_and_forms_beyond_it(torch_cuda, case, prism):
    """Each wave of a batch against the oracle's march (8-point rule on every axis): to 1e-8 in all, and the
    first current above a tenth of its peak, which the excitation alone drives, to 1e-11."""
    from oracle import mot
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    U, V, W, n = 5, 4, 3, 40
    geo = dict(c_dt=0.7, hy=0.7, hz=1.1) if prism else {}
    eps = wl.random_eps(U, V, W, 8, 1.0, 6.0)
    waves = []
    for sigma, k in CASES[case]:
        k = _unit(*k)
        p = np.cross(k, _unit(0.3, -0.5, 0.7))
        waves.append(wl.gaussian_wave(U, V, W, k, p / np.linalg.norm(p), sigma, 8.0 / sigma if sigma < 2 else 2.0))
    prob = wl.Problem(case, U, V, W, eps, waves, n, fir=wl.binomial_highpass(3, 0.01), **geo)
    print(case, prism, flush=True)
    s = motjvie.solver_for(prob)
    J = torch.zeros((n, len(waves), 3, W, V, U), dtype=torch.float64, device="cuda")
    s.run(n, J)
    s.close()
    J = J.cpu().numpy()
    K = None
    for r in range(len(waves)):
        one = wl.Problem("one", U, V, W, eps, [waves[r]], n, fir=prob.fir, **geo)
        o = mot.Oracle(one, K=K)
        K = o.K
        ref = o.run(n)
        assert np.linalg.norm(J[:, r] - ref) <= 1e-8 * np.linalg.norm(ref), r
        size = np.abs(ref).reshape(n, -1).max(axis=1)
        t = int(np.argmax(size >= 0.1 * size.max()))
        assert np.linalg.norm(J[t, r] - ref[t]) <= 1e-11 * np.linalg.norm(ref[t]), r

def test_pulse_far_narrower_than_a_voxel(torch_cuda):
    """A pulse of 1e-60 voxels, whose series does not exist in any number format: the average is what the pulse
    covers of a voxel, nothing beside its peak."""
    from paper_2407_03323_amd import motjvie
    U, V, W, n = 5, 4, 3, 8
    waves = [wl.PlaneWave(khat=k, pol=(0.0, 0.0, 1.0), width=1e-60, t0=0.5, amp=1.0, r_ref=(0.0, 0.0, 0.0))
             for k in ((1.0, 0.0, 0.0), (0.6, 0.8, 0.0))]   # the first passes a voxel's centre at every step
    prob = wl.Problem("narrow", U, V, W, wl.random_eps(U, V, W, 8, 2.0, 6.0), waves, n)
    s = motjvie.solver_for(prob)
    J = torch_cuda.zeros((n, 2, 3, W, V, U), dtype=torch_cuda.float64, device="cuda")
    s.run(n, J)
    s.close()
    assert float(J.abs().max()) <= 1e-50
