"""3D calls on an image of more rows than one dimension of a grid holds, against
the same image cut where no ray crosses the cut: with bins that reach the middle
rows only, the outer rows of a back-projection are zero and the middle ones those
of a small image (the same rays through the same voxels)."""
import numpy as np
import pytest

from tests.test_gpu_parity import dev, f32, host, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def desc(ny):
    return dict(dim=3, nx=6, ny=ny, nz=33, vx=2.0, vy=2.0, vz=2.5, n_angles=2, n_radial=301, ds=2.0, n_rings=33,
                max_ring_diff=1, ring_pitch=2.5, det_radius=1e5, n_subsets=1)


def test_back_projection_of_many_rows(orc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    big, small = pet.Geometry(desc(70001)), desc(401)
    # angle 0 runs along y, angle 1 (90 degrees) along x: only its bins, which
    # meet the 301 middle rows
    w = np.zeros(big.sino_shape, dtype=np.float32)
    w[:, 1, :] = f32(np.random.default_rng(3).uniform(0.5, 1.5, w[:, 1, :].shape))
    print("[gpu-many-rows]", flush=True)
    out = host(big.back(dev(w), 0))
    want = orc.back(orc.geom(small), w.astype(np.float64), 0)
    lo = (70001 - 401) // 2
    assert rel(out[:, lo:lo + 401], want) <= 1e-5
    assert not out[:, :lo].any() and not out[:, lo + 401:].any()
