"""The rounding of 3D back-projections on quads of mirror rays: no further from
the FP64 oracle than the column tiles were on the same kind of input (random
weights of one sign, 10 to 16 angles).  Both lane counts, four and five blocks
per CU, and chunks whose angles are no multiple of the groups summed together.

Tolerance: relative L2 of 1.0e-7.  FP32 sums of n positive terms in one chain err
by about 0.5 eps sqrt(n / 3) of their size, eps = 6e-8; a group of four angles
with up to 16 magnitudes and two bins each has n <= 128 in two chains, so about
1.5e-7 / sqrt(2) at its longest, and the rounding of the lengths (two roundings
of 0.3 eps each, independent over the terms) is small beside it.  One chain
through all angles measured 1.2e-7 to 1.7e-7."""
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


# nx, ny, nz, angles, bins, ring differences, subsets
@pytest.mark.parametrize("shape", [(64, 61, 29, 90, 93, 9, 9), (100, 97, 24, 84, 143, 7, 6), (60, 59, 64, 64, 87, 15, 4),
                                   (50, 52, 40, 90, 75, 11, 9), (200, 199, 9, 40, 285, 7, 4), (64, 64, 32, 48, 93, 15, 3)])
def test_error_against_64_bits(pet, orc, shape):
    nx, ny, nz, na, nr, rd, M = shape
    v = 300.0 / max(nx, ny)
    d = dict(dim=3, nx=nx, ny=ny, nz=nz, vx=v, vy=v, vz=3.0, n_angles=na, n_radial=nr, ds=v, n_rings=nz, max_ring_diff=rd,
             ring_pitch=3.0, det_radius=366.7, n_subsets=M)
    G, g = pet.Geometry(d), orc.geom(d)
    w = f32(np.random.default_rng(8).uniform(0.5, 1.5, G.sino_shape))
    err = rel(host(G.back(dev(w), 2)), orc.back(g, w, 2))
    print(f"[gpu-back-rounding] {shape} {err:.2e}", flush=True)
    assert err <= 1.0e-7
