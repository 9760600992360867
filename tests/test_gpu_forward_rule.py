"""3D forward projections on both sides of the rule between the projector that
stages single columns and the one on quads of mirror rays (depth a multiple of
4, up to 5 ring differences above 32 slices, up to 1 below): projections and
objectives against the FP64 oracle, and, in geometries that the quad
back-projector does not take (bins too fine or too few for it, more than 64
slices), whose weights come from either, a batched request bit for bit the one
alone.

Tolerance: 1e-5 relative L2 per projection, 1e-6 per objective, as everywhere."""
import numpy as np
import pytest

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


P = dict(mode="P2", beta=0.1, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=1e3, lambda0=0.5, a=0.25, rho=2.2, delta1=0.1,
         delta2=1.6, nu1=0.6, nu2=1.25, J0=0, J1=1000)


def desc(nx, ny, nz, rd, ds=2.0, nr=31):
    return dict(dim=3, nx=nx, ny=ny, nz=nz, vx=2.0, vy=2.0, vz=2.5, n_angles=12, n_radial=nr, ds=ds, n_rings=nz,
                max_ring_diff=rd, ring_pitch=2.5, det_radius=150.0, n_subsets=3)


@pytest.mark.parametrize("nx,ny,nz,rd", [(20, 19, 64, 0), (19, 20, 36, 5), (20, 20, 36, 6), (21, 18, 37, 2), (70, 9, 40, 3),
                                         (9, 70, 32, 1), (20, 18, 32, 2), (17, 20, 4, 0), (16, 16, 1, 0)])
def test_projection_and_objective(pet, orc, nx, ny, nz, rd):
    d = desc(nx, ny, nz, rd)
    print(f"[gpu-forward-rule] {nx}x{ny}x{nz} to {rd}", flush=True)
    G, g = pet.Geometry(d), orc.geom(d)
    rng = np.random.default_rng(12)
    f = f32(rng.uniform(0.5, 2.0, G.img_shape))
    for subset in (0, 2):
        sub = [a for a in range(12) if subset == 0 or a % 3 == subset - 1]
        assert rel(host(G.forward(dev(f), subset))[:, sub], orc.forward(g, f, subset)[:, sub]) <= 1e-5, subset
    y, r = f32(rng.poisson(30.0, G.sino_shape)), f32(rng.uniform(1.0, 3.0, G.sino_shape))
    phi, po = G.objective(P, dev(f), dev(y), dev(r)), orc.objective(g, f, y, r, P["beta"], P["gamma_R"], P["eps"])
    assert abs(phi - po) <= 1e-6 * abs(po)


@pytest.mark.parametrize("nz,rd,ds,nr", [(32, 1, 1.2, 51), (32, 2, 1.2, 51), (30, 1, 1.2, 51), (36, 0, 2.0, 9),
                                         (37, 0, 2.0, 9), (66, 3, 2.0, 31)])
def test_batch_equals_alone_bitwise(pet, nz, rd, ds, nr):
    G = pet.Geometry(desc(18, 17, nz, rd, ds=ds, nr=nr))
    print(f"[gpu-forward-rule] batch {nz} slices to {rd}", flush=True)
    rng = np.random.default_rng(13)
    y, r = dev(rng.poisson(30.0, G.sino_shape)), dev(rng.uniform(1.0, 3.0, G.sino_shape))
    a = dev(rng.uniform(0.5, 2.0, G.img_shape))
    b, c = a.clone(), a.clone()
    pet.reconstruct(G, P, a, y, r, 2)
    pet.reconstruct_batch([G, G], [P, P], [b, c], [y, y], [r, r], [2, 2])
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
