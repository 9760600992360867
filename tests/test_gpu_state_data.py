"""What a 3D state reads of y and r: with more than 15 ring differences it keeps
no copy of them, so that new contents in the same buffers count at once; up to
15 its copy stays as documented until it sees other buffers."""
import pytest

from synth import configs, phantoms
from tests.test_gpu_boundary import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    pet.lib()
    return pet


@pytest.mark.parametrize("rd", [15, 16, 19])
def test_new_contents_of_the_same_buffers(pet, rd):
    d = configs.desc_3d(20, 22, 12, 31, 2.5, 3.0, 22, rd, 4)
    w = phantoms.make_3d(d, seed=19, n_ell=3, counts=1e6, bg_uniform=0.15, bg_scatter=0.15, scatter_sigma_bins=4.0)
    p = configs.params_3d(U=w.U)
    G = pet.Geometry(w.desc)
    y, r, f = dev(w.y), dev(w.r), dev(w.f0)
    y2 = 2.0 * y
    st = pet.State(G, p)
    st.subiteration(f, y, r)
    f1 = f.clone()
    keep = y.clone()
    y.copy_(y2)
    st.subiteration(f, y, r)
    want = {}
    for name, data in (("old", keep), ("new", y2)):
        fresh = pet.State(G, p)
        fresh.seek(0, 2)
        h = f1.clone()
        fresh.subiteration(h, data, r)
        want[name] = h
    assert not torch.equal(want["old"], want["new"])
    assert torch.equal(f, want["old" if rd <= 15 else "new"])
