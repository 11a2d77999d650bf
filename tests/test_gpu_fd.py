"""The HIP full-order heat solver reproduces the oracle's FP64 finite-
difference solver bit for bit (same operations in the same order, no fused
multiply-add) in 1D and 2D, with scalar and per-node diffusivity (GPU)."""
import numpy as np
import pytest

from oracle import heat
from workloads import rng

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_node", [False, True])
def test_fd1d_bit_exact(cuda, per_node):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(1)
    n, n_grid = 257, 3
    u0 = g.uniform(-1, 1, size=(n_grid, n))
    nu = g.uniform(0.1, 1.0, size=(n_grid, n) if per_node else n_grid)
    dx = 1.0 / (n - 1)
    dt = 0.2 * dx * dx
    u = torch.from_numpy(u0.copy()).to(cuda)
    crom.fd_heat(u, torch.from_numpy(np.ascontiguousarray(nu)).to(cuda), dx, dt, 37)
    for k in range(n_grid):
        ref = heat.fd_heat1d(u0[k], nu[k], dx, dt, 37)
        np.testing.assert_array_equal(u[k].cpu().numpy(), ref)


@pytest.mark.parametrize("per_node", [False, True])
def test_fd2d_bit_exact(cuda, per_node):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(2)
    nx, ny, n_grid = 65, 48, 2
    u0 = g.uniform(-1, 1, size=(n_grid, nx, ny))
    nu = g.uniform(0.1, 1.0, size=(n_grid, nx, ny) if per_node else n_grid)
    dx = 1.0 / 63
    dt = 0.2 * dx * dx
    u = torch.from_numpy(u0.copy()).to(cuda)
    crom.fd_heat(u, torch.from_numpy(np.ascontiguousarray(nu)).to(cuda), dx, dt, 21)
    for k in range(n_grid):
        ref = heat.fd_heat2d(u0[k], nu[k], dx, dt, 21)
        np.testing.assert_array_equal(u[k].cpu().numpy(), ref)


def test_fd2d_256_grid_mode_decay(cuda):
    """256 x 256 grid (the 2D heat workload's size): a discrete sine mode
    decays by its exact amplification factor."""
    import torch
    from paper_2206_02607_amd import crom
    n = 256
    dx = 1.0 / (n - 1)
    x = np.arange(n) * dx
    X, Y = np.meshgrid(x, x, indexing="ij")
    mu = 0.7
    dt = 0.2 * dx * dx / mu
    u0 = np.sin(2 * np.pi * X) * np.sin(3 * np.pi * Y)
    u = torch.from_numpy(u0[None].copy()).to(cuda)
    crom.fd_heat(u, torch.tensor([mu], dtype=torch.float64), dx, dt, 100)
    r = mu * dt / dx ** 2
    lam = 1 - 4 * r * (np.sin(2 * np.pi * dx / 2) ** 2 + np.sin(3 * np.pi * dx / 2) ** 2)
    np.testing.assert_allclose(u[0].cpu().numpy(), lam ** 100 * u0, rtol=0, atol=1e-12)


# tiles of 64 x 128 nodes: one tile (all substeps in one launch), its edges,
# two tiles in either direction, odd and even launch counts
@pytest.mark.parametrize("per_node", [False, True])
@pytest.mark.parametrize("nx,ny,n_grid,steps", [(1, 7, 2, 3), (3, 3, 1, 5), (17, 19, 3, 40), (64, 128, 2, 33),
                                                (65, 128, 1, 1), (64, 129, 2, 29), (130, 257, 2, 50),
                                                (200, 64, 5, 26)])
def test_fd2d_tiles_bit_exact(cuda, nx, ny, n_grid, steps, per_node):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(nx * 1000 + ny)
    u0 = g.uniform(-1, 1, size=(n_grid, nx, ny)) * 10.0 ** g.integers(-250, 3, size=(n_grid, nx, ny))
    nu = g.uniform(0.1, 1.0, size=(n_grid, nx, ny) if per_node else n_grid)
    dx = 1.0 / 126.7
    dt = 0.2 * dx * dx
    u = torch.from_numpy(u0.copy()).to(cuda)
    crom.fd_heat(u, torch.from_numpy(np.ascontiguousarray(nu)).to(cuda), dx, dt, steps)
    for k in range(n_grid):
        np.testing.assert_array_equal(u[k].cpu().numpy(), heat.fd_heat2d(u0[k], nu[k], dx, dt, steps))


@pytest.mark.parametrize("dx,amp", [(1e-3, 1e150), (0.1, 1e302), (1e-40, 1.0)])
def test_fd2d_overflow(cuda, dx, amp):
    """Unstable and huge fields: infinities and NaN where the plain
    evaluation has them, one tile (in place) and several."""
    import torch
    from paper_2206_02607_amd import crom
    for nx, ny in ((40, 50), (150, 90)):
        u0 = rng(5).uniform(-1, 1, size=(1, nx, ny)) * amp
        u0[0, :, ny // 2:] = 0.0
        dt = 40.0 * dx * dx
        u = torch.from_numpy(u0.copy()).to(cuda)
        crom.fd_heat(u, torch.ones(1, dtype=torch.float64, device=cuda), dx, dt, 90)
        with np.errstate(all="ignore"):
            ref = heat.fd_heat2d(u0[0], 1.0, dx, dt, 90)
        np.testing.assert_array_equal(u[0].cpu().numpy(), ref)


# one launch per substep: many small fields (from 1,024 tiles on), narrow ones,
# one or two substeps of several tiles; and the neighbours of each that tiles take
@pytest.mark.parametrize("per_node", [False, True])
@pytest.mark.parametrize("n_grid,nx,ny,steps", [(1536, 3, 2, 9), (1536, 5, 6, 8), (1024, 8, 8, 7), (1, 40000, 5, 12),
                                                (1, 130, 257, 1), (1, 130, 257, 2), (1, 130, 257, 3), (2, 64, 129, 2),
                                                (700, 1, 4, 33), (3, 64, 128, 1)])
def test_fd2d_routes_bit_exact(cuda, n_grid, nx, ny, steps, per_node):
    import torch
    from paper_2206_02607_amd import crom
    g = rng(nx * 1000 + ny + steps)
    u0 = g.uniform(-1, 1, size=(n_grid, nx, ny)) * 10.0 ** g.integers(-250, 3, size=(n_grid, nx, ny))
    nu = g.uniform(0.1, 1.0, size=(n_grid, nx, ny) if per_node else n_grid)
    dx = 1.0 / 126.7
    dt = 0.2 * dx * dx
    u = torch.from_numpy(u0.copy()).to(cuda)
    crom.fd_heat(u, torch.from_numpy(np.ascontiguousarray(nu)).to(cuda), dx, dt, steps)
    got = u.cpu().numpy()
    for k in range(0, n_grid, max(1, n_grid // 50)):
        np.testing.assert_array_equal(got[k], heat.fd_heat2d(u0[k], nu[k], dx, dt, steps))


def test_fd2d_small_fields_cost(cuda):
    """A substep of many small fields is a pass over their memory, not a
    workgroup's tile for each: at most 2.5 times a copy (about 1.3)."""
    import torch
    from paper_2206_02607_amd import crom
    u = torch.rand(16384, 16, 16, dtype=torch.float64, device=cuda)
    v, nu, steps = torch.empty_like(u), torch.ones(16384, dtype=torch.float64, device=cuda), 40

    def us(f, n):
        best = 1e30
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(n):
                f()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1e3 / n)
        return best

    sub, copy = us(lambda: crom.fd_heat(u, nu, 0.01, 1e-6, steps, v), 2) / steps, us(lambda: v.copy_(u), steps)
    print(f"substep {sub:.1f} us, copy {copy:.1f} us")
    assert sub < 2.5 * copy, (sub, copy)
