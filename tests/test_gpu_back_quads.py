"""3D back-projections of weights in the natural layout go by quads of mirror
rays once the weights are many: against the FP64 oracle over the edges of the
layout (bins and sides odd and even, axis-parallel rays, depths at the ends of
the lane counts, bins too fine for it, few and many weights, more angles than a
run of quads), without a wait between calls on two streams, replayed under
capture, and with a weight that is not finite, which reaches only the voxels
that its LOR crosses.

Tolerance: 1e-5 relative L2, as for every projection."""
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


def desc(nx, ny, nz, na, nr, rd, M, ds=2.0):
    return dict(dim=3, nx=nx, ny=ny, nz=nz, vx=2.0, vy=2.0, vz=2.5, n_angles=na, n_radial=nr, ds=ds, n_rings=nz,
                max_ring_diff=rd, ring_pitch=2.5, det_radius=150.0, n_subsets=M)


@pytest.mark.parametrize("shape", [
    (20, 18, 32, 12, 31, 7, 3), (21, 19, 33, 12, 32, 5, 2), (17, 22, 64, 10, 34, 3, 1), (37, 35, 9, 40, 57, 8, 2),
    (18, 17, 20, 12, 47, 4, 1, 1.42), (18, 17, 20, 24, 55, 4, 1, 1.2), (16, 15, 64, 160, 25, 31, 1),
    (13, 12, 5, 4, 21, 1, 2)])
def test_natural_weights_match_the_oracle(pet, orc, shape):
    d = desc(*shape)
    print(f"[gpu-back-quads] {shape}", flush=True)
    G, g = pet.Geometry(d), orc.geom(d)
    w = f32(np.random.default_rng(6).uniform(-1.0, 1.0, G.sino_shape))
    for subset in {0, d["n_subsets"]}:
        assert rel(host(G.back(dev(w), subset)), orc.back(g, w, subset)) <= 1e-5, subset


def test_streams_and_capture(pet):
    G = pet.Geometry(desc(24, 23, 32, 12, 37, 7, 2))
    w = [torch.rand(G.sino_shape, device="cuda") for _ in range(2)]
    want = [G.back(x, 0) for x in w]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[torch.empty(G.img_shape, device="cuda") for _ in range(10)] for _ in w]
    torch.cuda.synchronize()
    for n in range(10):                     # no wait between the calls
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                G.back(w[i], 0, out=outs[i][n])
    torch.cuda.synchronize()
    assert all(torch.equal(o, want[i]) for i in (0, 1) for o in outs[i])
    x, out = w[0].clone(), torch.empty(G.img_shape, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        G.back(x, 0, out=out)
    for i in (0, 1, 0):
        x.copy_(w[i])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.allclose(out, want[i], rtol=1e-5, atol=1e-5 * float(want[i].max()))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_weight_that_is_not_finite_stays_on_its_lor(pet, bad):
    d = desc(24, 23, 32, 12, 37, 7, 1)      # angles 0 and 6: axis-parallel
    G = pet.Geometry(d)
    w = torch.rand(G.sino_shape, device="cuda")
    clean = G.back(w, 0)
    planes = G.sino_shape[0]
    for plane, a, b in ((0, 0, 18), (40, 0, 20), (planes - 1, 6, 10), (100, 3, 18), (200, 5, 30), (planes // 2, 1, 7)):
        one = torch.zeros_like(w)
        one[plane, a, b] = 1.0
        crossed = G.back(one, 0) > 0
        x = w.clone()
        x[plane, a, b] = bad
        out = G.back(x, 0)
        assert bool(torch.isfinite(out)[~crossed].all()), (plane, a, b)
        assert torch.equal(out[~crossed], clean[~crossed]), (plane, a, b)
        assert not bool(torch.isfinite(out)[crossed].any()), (plane, a, b)
