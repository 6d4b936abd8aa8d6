"""Every length of the two-radix FFT passes, along x, y and z, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [N for N in range(32, 257, 2)
         if any(N % a == 0 and 2 <= N // a <= 16 for a in range(2, 17))]


def _smooth(n):
    for p in (2, 3, 5, 7, 11, 13):
        while n % p == 0:
            n //= p
    return n == 1


SIZES = [N for N in SIZES if _smooth(N)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


# 3 and 17 x frequencies (one tile with idle pencils; a full tile and one pencil), pencils as picked and 5
@pytest.mark.parametrize("U,cap", [(2, 0), (16, 5)])
def test_two_radix_lengths(torch_cuda, U, cap):
    from paper_2407_03323_amd import motjvie
    torch = torch_cuda
    assert len(SIZES) == 49
    for i, Ny in enumerate(SIZES):
        Nz = SIZES[(i * 11 + 5) % len(SIZES)]
        if U > 2 and i % 4:
            continue
        V, W = Ny // 2, Nz // 2
        s = motjvie.Solver(U, V, W, np.full((W, V, U), 2.0), quad_order=4, fft_pencils=cap, time_block=1)
        info = s.info()
        assert (info["Ny"], info["Nz"]) == (Ny, Nz)
        _check(torch, s, info, (U, V, W))
        s.close()


@pytest.mark.parametrize("V,W,cap", [(2, 1, 0), (3, 5, 3)])
def test_two_radix_lengths_along_x(torch_cuda, V, W, cap):
    """Few rows (6: a tile with idle pencils) and an odd number of them (45: the last pencil holds one)."""
    from paper_2407_03323_amd import motjvie
    for i, Nx in enumerate(SIZES):
        if cap and i % 3:
            continue
        U = Nx // 2
        s = motjvie.Solver(U, V, W, np.full((W, V, U), 2.0), quad_order=4, fft_pencils=cap, time_block=1)
        info = s.info()
        assert info["Nx"] == Nx
        _check(torch_cuda, s, info, (U, V, W))
        s.close()


def _check(torch, s, info, UVW):
    U, V, W = UVW
    Ny, Nz = info["Ny"], info["Nz"]
    rng = np.random.default_rng(Ny)
    x = rng.standard_normal((3, W, V, U))
    xd = torch.tensor(x, device="cuda")
    X = torch.zeros((3, Nz, Ny, info["Nx"] // 2 + 1, 2), dtype=torch.float64, device="cuda")
    y = torch.zeros_like(xd)
    s.fft_roundtrip(xd, X, y)
    ref = np.fft.rfftn(x, s=(Nz, Ny, info["Nx"]), axes=(1, 2, 3))
    got = X.cpu().numpy()
    got = got[..., 0] + 1j * got[..., 1]
    # a few units in the last place per radix stage (three axes, two or more stages each)
    assert np.linalg.norm(got - ref) <= 2e-15 * np.linalg.norm(ref), (info["Nx"], Ny, Nz)
    back = y.cpu().numpy() / (info["Nx"] * Ny * Nz)
    assert np.linalg.norm(back - x) <= 2e-15 * np.linalg.norm(x), (info["Nx"], Ny, Nz)


# the shortest lengths, where a radix is 2 or 3; one of 6 points (no two-radix pass) beside them
@pytest.mark.parametrize("N", [6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 26, 28, 30])
@pytest.mark.parametrize("cap", [0, 3])
def test_short_lengths(torch_cuda, N, cap):
    from paper_2407_03323_amd import motjvie
    for U, V, W in ((N // 2, 5, 4), (4, N // 2, 3), (3, 4, N // 2)):
        s = motjvie.Solver(U, V, W, np.full((W, V, U), 2.0), quad_order=4, fft_pencils=cap, time_block=1)
        info = s.info()
        assert (info["Nx"], info["Ny"], info["Nz"]) == (2 * U, 2 * V, 2 * W)
        _check(torch_cuda, s, info, (U, V, W))
        s.close()
