"""3D forward projections of an image with a voxel that is not finite (a plain
projection does not check its image): every ray that crosses the voxel gives
what the sum over its pieces gives, an infinity or NaN, and the other rays keep
their bits.  Both lane counts of the quad projector, few and many ring
differences (the waves that share a magnitude's pieces), and a volume that it
does not take."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    pet.lib()
    return pet


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("shape", [(24, 23, 32, 7), (25, 22, 20, 12), (22, 24, 40, 15), (23, 21, 33, 1), (12, 11, 66, 3)])
def test_a_voxel_that_is_not_finite_stays_on_its_rays(pet, shape, bad):
    nx, ny, nz, rd = shape
    print(f"[gpu-forward-nonfinite] {shape} {bad}", flush=True)
    # 12 angles (0 and 6 axis-parallel)
    G = pet.Geometry(dict(dim=3, nx=nx, ny=ny, nz=nz, vx=2.0, vy=2.0, vz=2.5, n_angles=12, n_radial=37, ds=2.0, n_rings=nz,
                          max_ring_diff=rd, ring_pitch=2.5, det_radius=150.0, n_subsets=2))
    f = torch.rand(G.img_shape, device="cuda") + 0.5
    clean = G.forward(f, 0)
    for z, y, x in ((0, ny // 2, nx // 2), (nz // 2, 3, 5), (nz - 1, ny - 1, 0), (nz // 3, ny // 2, 1), (1, 0, nx - 1)):
        one = torch.zeros_like(f)
        one[z, y, x] = 1.0
        crossed = G.forward(one, 0) > 0
        g = f.clone()
        g[z, y, x] = bad
        q = G.forward(g, 0)
        assert torch.equal(q[~crossed], clean[~crossed]), (z, y, x)
        want = torch.full_like(q[crossed], bad)
        assert torch.equal(torch.nan_to_num(q[crossed], nan=7.0), torch.nan_to_num(want, nan=7.0)), (z, y, x)
