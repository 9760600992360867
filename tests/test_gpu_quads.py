"""3D projectors on quads of mirror rays against the FP64 oracle, where the
mirror symmetry has its edges: bins and image sides odd and even (a centre bin
that is its own mirror, a centre column that is its own mirror, axis-parallel
rays on cell edges), bins as fine as the quads allow and finer (the other
back-projector), anisotropic voxels, depths at the ends of the lane counts
(32, 33, 64 and beyond), no oblique planes and more magnitudes than a block or
a piece list holds.

Tolerance: 1e-5 relative L2 per projection, as for every projection; the
subset gradient within 1e-5 of its magnitude bound."""
import numpy as np
import pytest

from tests.test_gpu_gradcons import magnitude_bound
from tests.test_gpu_parity import dev, f32, host, rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    pet.lib()
    return pet


# nx, ny, nz, vx, vy, angles, bins, ds, ring differences, subsets
SHAPES = {
    "odd_centre_column": (21, 19, 9, 2.0, 2.0, 12, 33, 2.0, 3, 4),
    "even_edges_odd_bins": (20, 18, 32, 2.0, 2.0, 12, 31, 2.0, 7, 3),
    "even_edges_even_bins": (20, 18, 33, 2.0, 2.0, 12, 32, 2.0, 5, 3),
    "odd_edges_even_bins": (17, 22, 64, 2.0, 2.0, 10, 34, 2.0, 2, 5),
    "finest_bins": (18, 17, 20, 2.0, 2.0, 12, 47, 1.42, 4, 3),
    "finer_bins": (18, 17, 20, 2.0, 2.0, 12, 55, 1.2, 4, 3),
    "anisotropic": (15, 26, 40, 2.6, 1.9, 14, 37, 2.1, 6, 7),
    "direct_planes": (19, 16, 7, 2.0, 2.0, 9, 27, 2.0, 0, 2),
    "one_slice": (16, 16, 1, 2.0, 2.0, 8, 25, 2.0, 0, 2),
    "many_magnitudes": (16, 15, 50, 2.0, 2.0, 8, 25, 2.0, 31, 4),
    "full_obliqueness": (16, 15, 12, 2.0, 2.0, 8, 24, 2.0, 11, 4),
    "deeper_than_a_wave": (14, 13, 66, 2.0, 2.0, 6, 21, 2.0, 5, 3),
    "many_angles": (13, 12, 10, 2.0, 2.0, 70, 21, 2.0, 3, 2),
    "few_bins": (24, 24, 12, 2.0, 2.0, 12, 5, 2.0, 3, 3),
}


def desc(name):
    nx, ny, nz, vx, vy, na, nr, ds, rd, M = SHAPES[name]
    return dict(dim=3, nx=nx, ny=ny, nz=nz, vx=vx, vy=vy, vz=2.5, n_angles=na, n_radial=nr, ds=ds, n_rings=nz,
                max_ring_diff=rd, ring_pitch=2.5, det_radius=150.0, n_subsets=M)


@pytest.mark.parametrize("name", list(SHAPES))
def test_projections_and_gradient(pet, orc, name):
    from oracle import gradcons as gc
    d = desc(name)
    print(f"[gpu-quads] {name}", flush=True)
    G, g = pet.Geometry(d), orc.geom(d)
    rng = np.random.default_rng(4)
    f = f32(rng.uniform(0.5, 2.0, G.img_shape))
    y = f32(rng.poisson(30.0, G.sino_shape))
    r = f32(rng.uniform(1.0, 3.0, G.sino_shape))
    M = d["n_subsets"]
    p = dict(mode="P2", beta=0.1, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=1e3, lambda0=1.0, a=0.25, rho=2.2, delta1=0.1,
             delta2=1.6, nu1=0.6, nu2=1.25, J0=0, J1=1000)
    for subset in (0, 1, M):
        sel = gc._subset_rows(g, subset)
        assert rel(host(G.forward(dev(f), subset))[sel], orc.forward(g, f, subset)[sel]) <= 1e-5
        ho = gc.subset_gradient(g, f, y, r, subset, p["beta"], p["gamma_R"], p["eps"])
        hg = host(G.subset_gradient(p, dev(f), dev(y), dev(r), subset))
        bound = magnitude_bound(orc, g, f, y, r, subset, p)
        assert np.linalg.norm(hg - ho) <= 1e-5 * np.linalg.norm(bound), subset
    phi, po = G.objective(p, dev(f), dev(y), dev(r)), orc.objective(g, f, y, r, p["beta"], p["gamma_R"], p["eps"])
    assert abs(phi - po) <= 1e-6 * abs(po)


@pytest.mark.parametrize("name", ["even_edges_odd_bins", "even_edges_even_bins", "finer_bins", "many_magnitudes"])
def test_batch_equals_alone_bitwise(pet, name):
    """A batched request takes the projectors that it takes alone (both lane
    counts, either back-projector, the batch's own wave count)."""
    d = desc(name)
    G = pet.Geometry(d)
    rng = np.random.default_rng(5)
    y, r = dev(rng.poisson(30.0, G.sino_shape)), dev(rng.uniform(1.0, 3.0, G.sino_shape))
    f0 = dev(rng.uniform(0.5, 2.0, G.img_shape))
    p = dict(mode="P2", beta=0.1, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=1e3, lambda0=0.5, a=0.25, rho=2.2, delta1=0.1,
             delta2=1.6, nu1=0.6, nu2=1.25, J0=0, J1=1000)
    a, b, c = f0.clone(), f0.clone(), f0.clone()
    print(f"[gpu-quads] batch {name}", flush=True)
    pet.reconstruct(G, p, a, y, r, 2)
    pet.reconstruct_batch([G, G], [p, p], [b, c], [y, y], [r, r], [2, 2])
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
