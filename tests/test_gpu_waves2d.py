"""2D images of more 8x8 tiles than the device runs blocks at a time are
back-projected by a wave per tile: against the FP64 oracle, weights in either
layout, for ragged sides, angles in one chunk and several, axis-parallel rays,
windows of two bins and of more, and rays that miss the detector (few bins);
and with windows too wide for a wave, which keep a block per tile.

Tolerance: 1e-5 relative L2 per projection, as for every projection; the
subset gradient within 1e-5 of its magnitude bound."""
import numpy as np
import pytest

from tests.test_gpu_gradcons import magnitude_bound
from tests.test_gpu_parity import dev, f32, host, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx, ny, angles, bins, ds", [
    (257, 264, 8, 381, 2.0),        # 33 x 33 tiles: an odd last row and column
    (300, 301, 36, 429, 2.0),       # 18 angles: two chunks
    (312, 280, 6, 300, 2.0),        # corners outside the detector
    (280, 297, 6, 801, 1.05),       # three bins and more
    (272, 272, 4, 1500, 0.5),       # beyond a wave's staging
])
def test_wave_tiles_match_the_oracle(orc, nx, ny, angles, bins, ds):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    from oracle import gradcons as gc
    print(f"[gpu-waves2d] {nx}x{ny}", flush=True)
    d = dict(dim=2, nx=nx, ny=ny, nz=1, vx=2.0, vy=2.0, vz=1.0, n_angles=angles, n_radial=bins, ds=ds, n_rings=1,
             max_ring_diff=0, ring_pitch=1.0, det_radius=0.0, n_subsets=2)
    G, g = pet.Geometry(d), orc.geom(d)
    rng = np.random.default_rng(3)
    f = f32(rng.uniform(0.5, 2.0, G.img_shape))
    y = f32(rng.poisson(30.0, G.sino_shape))
    r = f32(rng.uniform(1.0, 3.0, G.sino_shape))
    p = dict(mode="P2", beta=0.1, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=1e3, lambda0=1.0, a=0.25, rho=2.2, delta1=0.1,
             delta2=1.6, nu1=0.6, nu2=1.25, J0=0, J1=1000)
    for subset in (0, 2):
        assert rel(host(G.back(dev(y), subset)), orc.back(g, y, subset)) <= 1e-5, subset
        ho = gc.subset_gradient(g, f, y, r, subset, p["beta"], p["gamma_R"], p["eps"])
        hg = host(G.subset_gradient(p, dev(f), dev(y), dev(r), subset))
        assert np.linalg.norm(hg - ho) <= 1e-5 * np.linalg.norm(magnitude_bound(orc, g, f, y, r, subset, p)), subset
