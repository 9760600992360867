"""3D back-projections on one stream while another is being captured: the
capture goes on, its graph replays what it recorded, and the back-projections
are those of any other time (rounding apart: one may take the kernel that needs
no scratch)."""
import pytest

from tests.test_gpu_back_quads import desc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_back_projection_beside_a_capture():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    G = pet.Geometry(desc(24, 23, 32, 12, 37, 7, 2))
    w = torch.rand(G.sino_shape, device="cuda")
    want = G.back(w, 0)
    outs = [torch.zeros(G.img_shape, device="cuda") for _ in range(6)]
    x = torch.zeros(1000, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    print("[gpu-beside-capture]", flush=True)
    with torch.cuda.graph(graph):
        x.add_(1.0)
        for o in outs:
            G.back(w, 0, out=o, stream=side)
        x.mul_(2.0)
    side.synchronize()
    for o in outs:
        assert torch.allclose(o, want, rtol=1e-5, atol=1e-5 * float(want.max()))
    for n in range(3):
        x.fill_(float(n))
        graph.replay()
        torch.cuda.synchronize()
        assert bool((x == 2.0 * (n + 1.0)).all())
