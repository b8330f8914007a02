"""Kernels at the sizes where their tiling can go wrong (block edges, remainders, list
capacities), against the float64 oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_density import _check_densify

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_05216_amd as P
    return P


@pytest.fixture(scope="module")
def ctx(P):
    return P.Context(0)


# ---------------------------------------------------------------- densify
@pytest.mark.parametrize("n,deg,n_split", [
    (1024, 3, 8),      # one block, far more outputs than one run of it holds
    (2049, 0, 8),      # the fewest rows, a one-Gaussian last block
    (5000, 1, 5)])
def test_densify_many_children(P, ctx, n, deg, n_split):
    from paper_2509_05216_amd import density as D
    ri = _check_densify(P, D, ctx, n, deg, 31 + n, 20.0, n_split)
    assert ri["children"] > 0


# ---------------------------------------------------------------- extraction
def _volume(kind, shape):
    nx, ny, nz = shape
    z, y, x = np.meshgrid(*(np.linspace(-1, 1, m) for m in (nz, ny, nx)), indexing="ij")
    if kind == "sphere":
        return (1.1 - np.sqrt(x * x + y * y + z * z)).astype(np.float32)
    v = np.random.default_rng(nx).random((nz, ny, nx)).astype(np.float32)
    if kind == "checker":   # every edge of the grid crosses
        i, j, k = np.meshgrid(*(np.arange(m) for m in (nz, ny, nx)), indexing="ij")
        return np.where((i + j + k) % 2 == 0, 0.2, 0.9).astype(np.float32) + 0.05 * v
    if kind == "ties":      # values on the level (never a crossing), NaN and infinities
        v = np.round(v * 4) / 4
        v.reshape(-1)[::7] = np.nan
        v.reshape(-1)[3::11] = np.inf
        v.reshape(-1)[5::13] = -np.inf
    return v.astype(np.float32)


@pytest.mark.parametrize("kind,shape,keep", [
    ("noise", (2, 3, 5000), 1.0), ("noise", (3, 5, 4), 0.5), ("noise", (4099, 3, 3), 1.0),
    ("noise", (2, 2049, 2), 1.0), ("checker", (33, 31, 29), 1.0), ("checker", (64, 64, 4), 0.25),
    ("ties", (40, 41, 13), 1.0),
    ("sphere", (263, 256, 257), 1.0)])    # more than 4096 blocks of 4096 vertices
def test_extraction_block_edges(P, ctx, kind, shape, keep):
    from oracle import iso as OI
    from paper_2509_05216_amd import iso
    vol = _volume(kind, shape)
    lo, hi = (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0)
    got = iso.extract(ctx, iso.Volume(torch.tensor(vol, device="cuda"), lo, hi), 0.5, keep, 9)
    got = got.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want, m = OI.extract(vol, lo, hi, 0.5, keep, 9)
    assert m > 0 and got.shape == want.shape
    # float64 positions rounded once: within one float32 ulp
    both = np.isfinite(want)
    assert np.array_equal(both, np.isfinite(got))
    ulp = np.spacing(np.abs(want[both]).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(got[both].astype(np.float64) - want[both]) <= ulp)
