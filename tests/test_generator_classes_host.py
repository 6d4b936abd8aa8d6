"""The generator's orders by distance and its stored offsets on the host (no GPU): the quadrature that the
device's kernels take with quad_order 0 against 16 points everywhere, and the permutations of an offset."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
DP, IP = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_int)


@pytest.fixture(scope="module")
def lib():
    out_dir = os.path.join(HERE, ".cache")
    os.makedirs(out_dir, exist_ok=True)
    so = os.path.join(out_dir, "libgen_classes.so")
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    cmd = [hipcc, "-O2", "-std=c++20", "-fPIC", "-shared", "-x", "hip", "--offload-arch=gfx950",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2407_03323_amd", "csrc"),
           os.path.join(HERE, "host", "gen_classes.cpp"), "-o", so]
    subprocess.check_call(cmd, stderr=subprocess.DEVNULL)
    L = ctypes.CDLL(so)
    L.host_class_kernels.argtypes = [DP, ctypes.c_double, ctypes.c_double, ctypes.c_double, ctypes.c_int,
                                     ctypes.c_int, DP]
    L.host_stored_offset.argtypes = [IP, IP, IP, DP]
    return L


def _kernels(L, D, r, hv, order):
    far = np.sqrt(sum(((abs(d) + 1) * h) ** 2 for d, h in zip(D, hv)))
    kmax = int(far / r) + 3
    D = np.ascontiguousarray(D, dtype=np.float64)
    out = np.zeros((kmax + 1, 6))
    cls = L.host_class_kernels(D.ctypes.data_as(DP), r, hv[1], hv[2], order, kmax, out.ctypes.data_as(DP))
    return cls, out


EDGES = [((1.0, 1.0, 1.0), 1.0), ((1.0, 1.0, 1.0), 0.45), ((1.0, 0.7, 1.3), 0.7), ((1.0, 1.0, 0.6), 0.55)]


@pytest.mark.parametrize("hv,r", EDGES)
def test_orders_by_distance_match_16_points(lib, hv, r):
    """Offsets of every class, on the grid and off it, in every octant: to the rounding of the sums (1e-14 to
    1e-13 of the offset's largest kernel; 1e-12 with a margin)."""
    rng = np.random.default_rng(7)
    seen = set()
    for i in range(150):
        D = rng.normal(size=3)
        D *= np.exp(rng.uniform(np.log(0.5), np.log(60.0))) / np.linalg.norm(D)
        if i % 3 == 0:
            D = np.round(D)
        cls, a = _kernels(lib, D, r, hv, 0)
        _, b = _kernels(lib, D, r, hv, 16)
        seen.add(cls)
        assert np.abs(b).max() > 0 and np.abs(a - b).max() <= 1e-12 * np.abs(b).max(), (D, cls)
    assert seen == set(range(5))


@pytest.mark.parametrize("hv,r", EDGES)
def test_grazing_spheres_match_16_points(lib, hv, r):
    """A sphere of the offset's shells cuts a plane of its squares in a circle between 1/1000 of a voxel and five
    of them, in front of the squares or beside them: as above."""
    rng = np.random.default_rng(11)
    for _ in range(150):
        ax = int(rng.integers(3))
        k = int(rng.integers(int(5.0 / r), int(40.0 / r)))
        rho = np.exp(rng.uniform(np.log(1e-3), np.log(5.0)))
        if rho >= k * r:
            continue
        c = np.sqrt((k * r) ** 2 - rho ** 2)
        D = np.zeros(3)
        D[ax] = c / hv[ax] + int(rng.integers(-1, 2))
        for o in (1, 2):
            D[(ax + o) % 3] = rng.uniform(0.0, 3.0)
        _, a = _kernels(lib, D, r, hv, 0)
        _, b = _kernels(lib, D, r, hv, 16)
        assert np.abs(b).max() > 0 and np.abs(a - b).max() <= 1e-12 * np.abs(b).max(), (D, rho)


@pytest.mark.parametrize("n", [(4, 4, 4), (5, 3, 4), (2, 5, 5), (1, 4, 3)])
@pytest.mark.parametrize("hv", [(1.0, 1.0, 1.0), (1.0, 1.0, 1.3), (1.0, 0.7, 1.0), (1.0, 0.7, 0.7), (1.0, 0.7, 1.3)])
def test_stored_offset_of_every_permutation(lib, n, hv):
    """The stored offset lies on the grid, is the offset with components traded along equal edges, and is the
    same for all of its permutations that the grid holds."""
    cn, ch = (ctypes.c_int * 3)(*n), (ctypes.c_double * 3)(*hv)

    def stored(d):
        cd, cp = (ctypes.c_int * 3)(*d), (ctypes.c_int * 3)()
        lib.host_stored_offset(cd, cp, cn, ch)
        return tuple(cd), tuple(cp)

    for d in itertools.product(*(range(k) for k in n)):
        s, pos = stored(d)
        assert sorted(pos) == [0, 1, 2] and all(0 <= s[i] < n[i] for i in range(3))
        assert all(s[pos[a]] == d[a] and hv[pos[a]] == hv[a] for a in range(3))
        assert stored(s) == (s, (0, 1, 2))
        for q in itertools.permutations(range(3)):
            if all(hv[q[a]] == hv[a] and d[q[a]] < n[a] for a in range(3)):
                assert stored(tuple(d[q[a]] for a in range(3)))[0] == s
