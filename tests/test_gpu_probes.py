"""Probe sums and adjoint sources taken several steps at a time."""
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


# windows of 5 to 12 lags (below and above the 8 steps of a launch), runs that end inside a group of steps,
# more and fewer pairs than a chunk's 128, and two right-hand sides
@pytest.mark.parametrize("UVW,r,nr", [((3, 2, 2), 1.0, 1), ((7, 6, 5), 0.7, 2), ((9, 8, 7), 0.35, 1)])
def test_probe_field_by_step_and_by_run(torch_cuda, UVW, r, nr):
    """One call a step, runs of 1, 2, 7, 8, 9, 16, 17 steps, and one run give the same field bit for bit, and
    it is the sum over the lags of the kernels the solver reports (64-bit sums in another order)."""
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    U, V, W = UVW
    n = 60
    eps = wl.random_eps(U, V, W, 3, 1.5, 9.0)
    waves = [wl.gaussian_wave(U, V, W, k, p, 2.0, 3.0) for k, p in wl.random_directions(nr, 4)]
    prob = wl.Problem("probes", U, V, W, eps, waves, n, fir=wl.binomial_highpass(3, 0.01), c_dt=r)
    pts = wl.fibonacci_sphere(3, 1.5 * max(UVW), (U / 2, V / 2, W / 2))
    out = []
    for parts in ([n], [1] * n, [1, 2, 7, 8, 9, 16, 17]):
        s = motjvie.solver_for(prob)
        s.set_probes(pts)
        J = torch.zeros((n, nr, 3, W, V, U), dtype=torch.float64, device="cuda")
        E = torch.zeros((n, nr, 3, 3), dtype=torch.float64, device="cuda")
        at = 0
        for m in parts:
            s.run(m, J[at:at + m], E[at:at + m])
            at += m
        out.append((J, E))
        if len(parts) == 1:
            ell, M = s.ell, U * V * W
            vox = [(u, v, w) for w in range(W) for v in range(V) for u in range(U)]
            K = np.stack([s.probe_kernel_values([p] * M * (ell + 1), vox * (ell + 1),
                                                np.repeat(np.arange(ell + 1), M)).reshape(ell + 1, M, 6)
                          for p in range(3)])
        s.close()
    assert all(torch.equal(out[0][1], e) and torch.equal(out[0][0], j) for j, e in out[1:])
    Jn = out[0][0].cpu().numpy().reshape(n, nr, 3, -1)
    K3 = K[..., [[0, 3, 4], [3, 1, 5], [4, 5, 2]]]
    ref = np.zeros((n, nr, 3, 3))
    for k in range(ell + 1):
        ref[k:] += np.einsum("pmba,nram->nrpb", K3[:, k], Jn[: n - k])
    got = out[0][1].cpu().numpy()
    assert np.abs(ref).max() > 0
    assert np.linalg.norm(got - ref) <= 1e-13 * np.linalg.norm(ref)


def test_state_between_probe_groups(torch_cuda):
    """A state taken inside a group of 8 steps, whose ring is shorter than the solver's, resumes the field
    bit for bit."""
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    U, V, W, n, m = 6, 5, 4, 50, 29
    eps = wl.random_eps(U, V, W, 41, 2.0, 9.0)
    k, p = wl.XPOL_PLUS_Z
    prob = wl.Problem("resume", U, V, W, eps, [wl.gaussian_wave(U, V, W, k, p, 2.0)], n)
    pts = wl.fibonacci_sphere(3, 5.0, (U / 2, V / 2, W / 2))
    s = motjvie.solver_for(prob)
    s.set_probes(pts)
    assert s.info()["real_depth"] == max(8, s.ell + 1)
    E = torch.zeros((n, 1, 3, 3), dtype=torch.float64, device="cuda")
    s.run(m, None, E[:m])
    st = s.get_state()
    s.run(n - m, None, E[m:])
    s.close()
    s = motjvie.solver_for(prob)
    s.set_probes(pts)
    s.set_state(st)
    F = torch.zeros((n - m, 1, 3, 3), dtype=torch.float64, device="cuda")
    s.run(n - m, None, F)
    s.close()
    assert float(E.norm()) > 0 and torch.equal(E[m:], F)


@pytest.fixture
def nan_memory(torch_cuda, monkeypatch):
    """The library's device memory filled with NaN before it gets it (allocator="torch")."""
    from paper_2407_03323_amd import motjvie
    torch, held = torch_cuda, {}

    def alloc(nbytes, ctx):
        t = torch.full(((int(nbytes) + 7) // 8,), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        held[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, ctx):
        torch.cuda.synchronize()
        del held[ptr]

    monkeypatch.setattr(motjvie, "torch_allocator", lambda stream: (motjvie.ALLOC_FN(alloc), motjvie.FREE_FN(free)))


# outside receivers, whose windows reach beyond the last lag: the steps those lags name are not in a state
@pytest.mark.parametrize("UVW,r,nr,radius", [((6, 5, 4), 1.0, 1, 5.0), ((7, 6, 5), 0.7, 2, 9.0)])
def test_resumed_probe_field_reads_the_state_alone(torch_cuda, nan_memory, UVW, r, nr, radius):
    """The first calls after mj_set_state, of 1, 2, 3 and 7 steps, repeat the uninterrupted march bit for bit in
    memory that held NaN: no sum reads a ring slot that the state does not fill."""
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    U, V, W = UVW
    m, more = 33, 7
    eps = wl.random_eps(U, V, W, 41, 2.0, 9.0)
    waves = [wl.gaussian_wave(U, V, W, k, p, 2.0, 3.0) for k, p in wl.random_directions(nr, 4)]
    prob = wl.Problem("resume", U, V, W, eps, waves, m + more, fir=wl.binomial_highpass(3, 0.01), c_dt=r)
    pts = wl.fibonacci_sphere(3, radius, (U / 2, V / 2, W / 2))
    s = motjvie.solver_for(prob)
    s.set_probes(pts)
    s.run(m)
    st = s.get_state()
    E = torch.zeros((more, nr, 3, 3), dtype=torch.float64, device="cuda")
    s.run(more, None, E)
    s.close()
    assert float(E.norm()) > 0
    for first in (1, 2, 3, 7):
        s = motjvie.solver_for(prob, allocator="torch")
        s.set_probes(pts)
        s.set_state(st)
        F = torch.zeros_like(E)
        s.run(first, None, F[:first])
        if first < more:
            s.run(more - first, None, F[first:])
        s.close()
        assert torch.equal(E, F), first


def test_probes_that_do_not_fit_leave_a_solver_without_them(torch_cuda, monkeypatch):
    """mj_set_probes out of memory at each of its allocations: MJ_ENOMEM, no probes, and the march, and probes
    that fit, work as in a solver that never met it."""
    from paper_2407_03323_amd import motjvie
    from paper_2407_03323_amd.motjvie import MJ_ENOMEM, MJ_ESTATE, MotJvieError
    torch, held, left = torch_cuda, {}, [10 ** 6]

    def alloc(nbytes, ctx):
        left[0] -= 1
        if left[0] < 0:
            return None
        t = torch.zeros(((int(nbytes) + 7) // 8,), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        held[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, ctx):
        torch.cuda.synchronize()
        del held[ptr]

    monkeypatch.setattr(motjvie, "torch_allocator", lambda stream: (motjvie.ALLOC_FN(alloc), motjvie.FREE_FN(free)))
    U, V, W, n = 6, 5, 4, 12
    k, p = wl.XPOL_PLUS_Z
    prob = wl.Problem("full", U, V, W, wl.random_eps(U, V, W, 41, 2.0, 9.0), [wl.gaussian_wave(U, V, W, k, p, 2.0, 2.0)], n)
    pts = wl.fibonacci_sphere(3, 5.0, (U / 2, V / 2, W / 2))

    def march(s):
        J = torch.zeros((n, 1, 3, W, V, U), dtype=torch.float64, device="cuda")
        s.reset()
        s.run(n, J)
        return J

    s = motjvie.solver_for(prob, allocator="torch")
    plain = march(s)
    s.reset()
    s.set_probes(pts)
    E = torch.zeros((n, 1, 3, 3), dtype=torch.float64, device="cuda")
    s.run(n, None, E)
    s.close()
    s = motjvie.solver_for(prob, allocator="torch")
    fits = 0
    while True:
        s.reset()
        left[0] = fits
        try:
            s.set_probes(pts)
        except MotJvieError as e:
            assert e.code == MJ_ENOMEM
        else:
            break
        finally:
            left[0] = 10 ** 6
        fits += 1
        assert s.info()["n_probes"] == 0
        with pytest.raises(MotJvieError) as ei:
            s.adjoint_gradient(n, torch.zeros((W, V, U), dtype=torch.float64, device="cuda"))
        assert ei.value.code == MJ_ESTATE
        assert torch.equal(march(s), plain)
    assert fits >= 10
    F = torch.zeros_like(E)
    s.run(n, None, F)
    s.close()
    assert torch.equal(E, F) and float(E.norm()) > 0 and not held
