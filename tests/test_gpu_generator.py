"""The kernel generator's order classes, its stored offsets and the cut edges of its squares, on the device
against the oracle's quadrature."""
import numpy as np
import pytest

from oracle import mot

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _solver(U, V, W, **kw):
    from paper_2407_03323_amd import motjvie
    return motjvie.Solver(U, V, W, np.full((W, V, U), 4.0), **kw)


# gaps on both sides of 3.5, 6, 12 and 24 edges, in every order of the axes that the box holds; axes of equal
# and unequal edges, as many and fewer voxels along the axis that takes the larger component
@pytest.mark.parametrize("UVW,hv,r", [((30, 9, 14), (1.0, 1.0, 1.0), 1.0), ((9, 30, 14), (1.0, 1.0, 1.3), 0.8),
                                      ((14, 9, 30), (1.0, 0.7, 1.0), 0.7)])
def test_order_classes_and_stored_offsets(torch_cuda, UVW, hv, r):
    U, V, W = UVW
    s = _solver(U, V, W, hy=hv[1], hz=hv[2], c_dt=r)
    print("classes", UVW, hv, r, flush=True)
    for d in [(4, 1, 0), (4, 2, 1), (5, 1, 2), (6, 3, 1), (7, 0, 0), (7, 2, 3), (8, 3, 0), (12, 3, 7), (13, 0, 1),
              (13, 8, 4), (24, 1, 0), (25, 2, 1), (27, 8, 5), (2, 2, 8)]:
        for perm in ((0, 1, 2), (1, 0, 2), (2, 1, 0), (0, 2, 1), (1, 2, 0), (2, 0, 1)):
            D = tuple(d[p] * sg for p, sg in zip(perm, (1, -1, 1)))
            if any(abs(x) >= n for x, n in zip(D, UVW)):
                continue
            far = np.sqrt(sum(((abs(x) + 1) * h) ** 2 for x, h in zip(D, hv)))
            near = np.sqrt(sum((max(abs(x) - 1, 0) * h) ** 2 for x, h in zip(D, hv)))
            lags = [k for k in range(int(near / r), int(far / r) + 3) if k <= s.ell]
            got = s.kernel_values(lags, [D] * len(lags))
            ref = np.array([mot.kernel_entry(k, D, ngl=16, r=r, hv=hv) for k in lags])
            assert np.abs(got - ref).max() <= 3e-12 * np.abs(ref).max(), (D, np.abs(got - ref).max())
    s.close()


def test_edges_cut_around_their_nearest_point(torch_cuda):
    """Probes whose squares straddle the foot of the perpendicular while the outer sphere just crosses
    their nearest edge on both sides of it: the interval between the crossings counts."""
    D = [(0.4928115528680801, 0.2451472281789438, 2.6486588989243938),
         (0.4290604436623726, 5.97884416415982, 5.185160847563338),
         (4.544344548265136, 1.936848053762032, 0.3305983516361867)]
    s = _solver(3, 3, 3, c_dt=0.45)
    s.set_probes(np.array(D) + 0.5)   # seen from voxel (0, 0, 0)
    for p, d in enumerate(D):
        n = 30   # lags that every one of these reaches
        got = s.probe_kernel_values([p] * n, [(0, 0, 0)] * n, list(range(n)))
        ref = np.array([mot.kernel_entry(k, d, ngl=24, r=0.45) for k in range(n)])
        assert np.abs(ref).max() > 0 and np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
    s.close()


@pytest.mark.parametrize("hv,r,D", [
    ((1.0, 0.7, 1.3), 0.7, [(13.595790667296122, 1.0400267473549167, 0.29396812422172935),
                            (13.595790667296122, 1.0400267473549167, 1.006031875778271),
                            (6.594792936872352, 1.0397363021375359, 0.2936997818765675),
                            (12.888234457101511, 1.2429470524374953, 0.16522220916036323)]),
    ((1.0, 1.0, 1.0), 1.0, [(9.0 + 1.0 - 0.004, 1.31, 0.22), (0.4, 14.0 - 0.006, 1.2), (1.25, 0.1, 30.0 - 0.003)]),
])
def test_spheres_that_graze_a_plane(torch_cuda, hv, r, D):
    """Far probes in front of a voxel whose plane a sphere cuts in a circle smaller than the voxel: the few
    points of their distance do not follow the rays there, and the shell takes 16.  Against 16 points
    everywhere, to the rounding of the sums (1e-13 at these distances; 1e-12 with a margin)."""
    out = []
    for q in (0, 16):
        s = _solver(3, 3, 3, hy=hv[1], hz=hv[2], c_dt=r, quad_order=q)
        s.set_probes(np.array(D) + 0.5 * np.array(hv))   # seen from voxel (0, 0, 0)
        n = 50   # beyond the last lag that reaches any of these
        out.append([s.probe_kernel_values([p] * n, [(0, 0, 0)] * n, list(range(n))) for p in range(len(D))])
        s.close()
    for a, b in zip(*out):
        assert np.abs(b).max() > 0 and np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
