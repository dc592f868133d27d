"""GPU parity of the 3-D diffusion step (section "3D diffusion equation")
against the FP64 oracle on the same FP32 grid. The update is a convex-ish
combination of seven FP32 values with FP32 coefficients: its rounding error
is a few ulps of max|f|, bound here by 1e-6 of max|f|."""

import numpy as np
import pytest
import torch

import oracle
import paper_2411_18889_amd as nb
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

PARAMS = dict(dx=0.5, dy=0.25, dz=1.0, dt=0.01, kappa=1.5)


def _check(f32):
    fd = torch.tensor(f32, device=DEV)
    fn = nb.api.diffusion3d_step(fd, **PARAMS).cpu().numpy().astype(np.float64)
    ref = oracle.diffusion3d(f32.astype(np.float64), **PARAMS)
    err = np.abs(fn - ref).max() / np.abs(ref).max()
    assert err <= 1e-6, err
    return fn, ref


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 5), (7, 9, 65), (33, 17, 130),
                                   (64, 64, 64), (40, 70, 129), (65, 8, 64)])
def test_random_grids(shape):
    f = np.random.default_rng(sum(shape)).uniform(-1, 1, size=shape).astype(np.float32)
    _check(f)


def test_cosine_mode_eigenvalue():
    shape = (48, 40, 96)
    nx, ny, nz = shape
    i = np.arange(nx)[:, None, None]
    j = np.arange(ny)[None, :, None]
    k = np.arange(nz)[None, None, :]
    p, q, r = 3, 5, 7
    f = (np.cos(np.pi * p * (i + 0.5) / nx) * np.cos(np.pi * q * (j + 0.5) / ny)
         * np.cos(np.pi * r * (k + 0.5) / nz)).astype(np.float32)
    fn, _ = _check(f)
    c = [PARAMS["kappa"] * PARAMS["dt"] / h ** 2 for h in (PARAMS["dx"], PARAMS["dy"], PARAMS["dz"])]
    lam = 1 - 4 * sum(ck * np.sin(np.pi * m / (2 * n)) ** 2 for ck, m, n in zip(c, (p, q, r), shape))
    assert np.abs(fn - lam * f).max() <= 1e-6


def test_paper_size_sampled_planes():
    """512^3 (the paper's best-performing size) in the launch shape the bench
    times; the oracle checks every point."""
    shape = (512, 512, 512)
    f = np.random.default_rng(5).uniform(0, 1, size=shape).astype(np.float32)
    _check(f)


def test_mass_conserved_on_gpu():
    f = np.random.default_rng(9).uniform(0, 1, size=(96, 80, 72)).astype(np.float32)
    fd = torch.tensor(f, device=DEV)
    fn = nb.api.diffusion3d_step(fd, **PARAMS)
    s0, s1 = float(fd.double().sum()), float(fn.double().sum())
    assert abs(s1 - s0) <= 1e-6 * s0


@pytest.mark.parametrize("shape", [(3, 5, 3), (1, 1, 2), (5, 1, 4), (1, 9, 5), (9, 3, 7), (2, 6, 8),
                                   (20, 33, 255), (18, 5, 257), (17, 31, 259), (300, 3, 9),
                                   (337, 317, 315), (130, 509, 508), (9, 2051, 2049)])
def test_ragged_rows(shape):
    """Row lengths around the 4 points of a lane and the 256 of a wave, rows
    shorter than a lane, slabs that end inside the grid; from the last-level
    cache's size on (the last three) four rows per lane, with rows left over.
    Unaligned input and output: both start one element into their storage."""
    n = int(np.prod(shape))
    f = np.random.default_rng(n).uniform(-1, 1, size=shape).astype(np.float32)
    fd = torch.empty(n + 1, dtype=torch.float32, device=DEV)[1:].view(shape)
    fd.copy_(torch.tensor(f))
    guard = torch.full((n + 2,), 7.0, dtype=torch.float32, device=DEV)
    fn = nb.api.diffusion3d_step(fd, out=guard[1:-1].view(shape), **PARAMS)
    ref = oracle.diffusion3d(f.astype(np.float64), **PARAMS)
    assert np.abs(fn.cpu().numpy() - ref).max() <= 1e-6 * np.abs(ref).max()
    assert float(guard[0]) == 7.0 and float(guard[-1]) == 7.0


@pytest.mark.parametrize("nz", (2 ** 31 - 1, 2 ** 31 - 3, 2 ** 31 - 4))
def test_longest_rows(nz):
    """One row of as many points as a grid may have, where 4 points a lane end
    past an int: every point against the update of the same FP32 values in
    FP64 (in pieces); j and i have no neighbours, so theirs are the point
    itself."""
    f = torch.empty(nz, dtype=torch.float32, device=DEV)
    torch.manual_seed(nz % 1000)
    f.uniform_(-1, 1)
    fn = nb.api.diffusion3d_step(f.view(1, 1, nz), **PARAMS).view(nz)
    ct = PARAMS["kappa"] * PARAMS["dt"] / PARAMS["dz"] ** 2
    for k0 in range(0, nz, 1 << 27):
        k1 = min(nz, k0 + (1 << 27))
        c = f[k0:k1].double()
        ref = c * (1 - 2 * ct)
        ref[1:] += ct * c[:-1]
        ref[:-1] += ct * c[1:]
        ref[0] += ct * f[max(k0 - 1, 0)].double()
        ref[-1] += ct * f[min(k1, nz - 1)].double()
        assert float((fn[k0:k1] - ref).abs().max()) <= 1e-6


@pytest.mark.parametrize("shape", [(131, 709, 507), (70, 1, 600001), (20, 250001, 7), (5, 5003, 1400),
                                   (33, 1025, 1024)])
def test_large_planes(shape):
    """Grids beyond the last-level cache whose planes do not fit an L2 three at a
    time: workgroups that keep pace by barriers, with lanes past the end of the
    plane, slabs that end inside the grid, rows of two lanes and single rows,
    unaligned input and output, and nothing written outside."""
    n = int(np.prod(shape))
    f = np.random.default_rng(n).uniform(-1, 1, size=shape).astype(np.float32)
    fd = torch.empty(n + 1, dtype=torch.float32, device=DEV)[1:].view(shape)
    fd.copy_(torch.tensor(f))
    guard = torch.full((n + 2,), 7.0, dtype=torch.float32, device=DEV)
    fn = nb.api.diffusion3d_step(fd, out=guard[1:-1].view(shape), **PARAMS)
    ref = oracle.diffusion3d(f.astype(np.float64), **PARAMS)
    assert np.abs(fn.cpu().numpy() - ref).max() <= 1e-6 * np.abs(ref).max()
    assert float(guard[0]) == 7.0 and float(guard[-1]) == 7.0
