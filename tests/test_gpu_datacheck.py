"""The data check reads its arrays 16 bytes at a time from their first aligned
element: bad values counted one by one at both ends and in the middle, for
arrays that start at each of the four positions in a 16-byte group and have
every remainder, and smaller than a group."""
import re

import pytest

from tests.test_gpu_boundary import small_2d

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("start", [0, 1, 2, 3])
@pytest.mark.parametrize("nx, bins, angles", [(4, 7, 2), (9, 13, 3), (33, 47, 11), (640, 905, 360)])
def test_bad_values_are_counted(nx, bins, angles, start):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    w, p = small_2d()
    d = dict(w.desc, nx=nx, ny=nx, n_angles=angles, n_radial=bins, n_subsets=1)
    G = pet.Geometry(d)

    def array(shape, v):
        n = shape[-1] * shape[-2]
        return torch.full((n + start,), v, device="cuda")[start:].view(shape)
    y, r, f = array(G.sino_shape, 3.0), array(G.sino_shape, 1.0), array(G.img_shape, 0.5 * p["U"])
    n = y.numel()
    places = sorted({0, 1, 2, 3, 4, n // 2, n - 5, n - 4, n - 3, n - 2, n - 1})
    for name, x, bad in (("y", y, float("nan")), ("r", r, 0.0), ("f", f, 2.0 * p["U"])):
        here = [q for q in places if 0 <= q < x.numel()]
        keep = x.clone()
        x.view(-1)[here] = bad
        with pytest.raises(pet.PetOSError) as e:
            pet.reconstruct(G, p, f, y, r, 1)
        assert re.search(rf"{name}: {len(here)} entries", str(e.value)), (name, len(here), str(e.value))
        x.copy_(keep)
