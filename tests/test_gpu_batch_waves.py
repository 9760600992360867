"""A batch of many 2D tiles takes a wave per 8x8 tile: bit for bit what each
request computes alone, for ragged images whose last block holds one, two or
three tiles, images smaller than a tile, axis-parallel angles, bins coarse and
fine (windows of more than two bins, and of more weights than a wave stages),
few angles and more than one chunk of them, and every mode."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# nx, ny, angles, bins, ds, subsets, mode
REQUESTS = [
    (300, 301, 40, 429, 2.0, 8, "P2"),      # 1444 tiles: the batch goes by waves
    (41, 55, 36, 71, 2.0, 2, "M1"),         # 18 angles: two chunks
    (7, 5, 12, 13, 2.0, 4, "P1"),           # less than a tile
    (17, 8, 9, 31, 2.0, 3, "BSREM"),        # a block of tiles in one row
    (64, 72, 20, 181, 1.1, 4, "M2"),        # windows of three bins and more
    (33, 24, 15, 201, 0.4, 5, "P2"),        # windows beyond a wave's staging
    (48, 48, 6, 25, 6.5, 2, "P2"),          # bins wider than three pixels
]


def test_batch_by_waves_equals_alone_bitwise():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    rng = np.random.default_rng(8)

    def dev(x):
        return torch.tensor(np.ascontiguousarray(x, dtype=np.float32), device="cuda")
    geoms, ps, ys, rs, fs, alone, iters = [], [], [], [], [], [], []
    for k, (nx, ny, na, nr, ds, M, mode) in enumerate(REQUESTS):
        print(f"[gpu-batch-waves] {nx}x{ny} alone", flush=True)
        G = pet.Geometry(dict(dim=2, nx=nx, ny=ny, nz=1, vx=2.0, vy=2.0, vz=1.0, n_angles=na, n_radial=nr, ds=ds,
                              n_rings=1, max_ring_diff=0, ring_pitch=1.0, det_radius=0.0, n_subsets=M))
        p = dict(mode=mode, beta=0.1, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=1e3, lambda0=0.5, a=0.25, rho=2.2,
                 delta1=0.1, delta2=1.6, nu1=0.6, nu2=1.25, J0=0, J1=3)
        y, r = dev(rng.poisson(30.0, G.sino_shape)), dev(rng.uniform(1.0, 3.0, G.sino_shape))
        f = dev(rng.uniform(0.5, 2.0, G.img_shape))
        x = f.clone()
        pet.reconstruct(G, p, x, y, r, 2 + k % 2)
        geoms.append(G), ps.append(p), ys.append(y), rs.append(r), fs.append(f), alone.append(x)
        iters.append(2 + k % 2)
    print("[gpu-batch-waves] batch", flush=True)
    pet.reconstruct_batch(geoms, ps, fs, ys, rs, iters)
    torch.cuda.synchronize()
    for k, (a, b) in enumerate(zip(alone, fs)):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b), REQUESTS[k]
