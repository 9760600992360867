"""Every shape of k_bp3 that the 3D autotuner can choose, pinned through its
cache file, in geometries whose subiterations use that kernel (more than 64
slices; bins too fine for quads): natural weights of one subset and of every
angle, and fused subiterations (compact weights, the penalty in the same launch)
against the oracle.  That k_bp3 is the back-projector in use is seen by the
autotuner, which times its shapes only then.

Tolerance: 1e-5 relative L2 per projection and per subiteration."""
import numpy as np
import pytest

from tests.test_gpu_parity import dev, f32, full_desc, host, rel, say, stepwise, tune_key

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    pet.lib()
    return pet


GEOMS = {
    "deep": dict(dim=3, nx=27, ny=21, nz=70, vx=2.0, vy=2.0, vz=2.5, n_angles=16, n_radial=39, ds=2.0, n_rings=70,
                 max_ring_diff=2, ring_pitch=2.5, det_radius=150.0, n_subsets=4),
    "fine_bins": dict(dim=3, nx=26, ny=23, nz=20, vx=2.0, vy=2.0, vz=2.5, n_angles=16, n_radial=53, ds=1.3, n_rings=20,
                      max_ring_diff=4, ring_pitch=2.5, det_radius=150.0, n_subsets=4),
}


@pytest.mark.parametrize("name,zb,dpg", [("deep", 16, 4), ("deep", 16, 8), ("deep", 32, 4), ("deep", 32, 8), ("deep", 64, 4),
                                         ("fine_bins", 16, 4), ("fine_bins", 32, 4)])
def test_shapes(pet, orc, tmp_path, monkeypatch, name, zb, dpg):
    from synth import configs, phantoms
    d = full_desc(GEOMS[name])
    cache = tmp_path / "tune.txt"
    cache.write_text(f"{tune_key(d)}|0 {zb * 16 + dpg}\n")
    monkeypatch.setenv("PET_OS_TUNE_CACHE", str(cache))
    say(f"bp3 shape {name} zb={zb} dpg={dpg}")
    G = pet.Geometry(d)
    pet.autotune(G, force=True)
    assert cache.read_text().count("|") == 2            # timed: subiterations use k_bp3
    cache.write_text(f"{tune_key(d)}|0 {zb * 16 + dpg}\n")
    pet.autotune(G)
    sh = G.shapes()
    assert (sh["current"]["bp3_zb"], sh["current"]["bp3_dpg"]) == (zb, dpg)
    g = orc.geom(d)
    rng = np.random.default_rng(zb + dpg)
    wv = f32(rng.uniform(-1.0, 1.0, G.sino_shape))
    assert rel(host(G.back(dev(wv), 2)), orc.back(g, wv, 2)) <= 1e-5
    ones = np.ones(G.sino_shape)
    assert rel(host(G.back(dev(ones), 0)), orc.back(g, ones, 0)) <= 1e-5
    w = phantoms.make_3d(d, seed=31, n_ell=4, counts=2e6, bg_uniform=0.15, bg_scatter=0.15, scatter_sigma_bins=4.0)
    stepwise(pet, orc, w, configs.params_3d(U=w.U), {1, 2, 5}, tune=True)
