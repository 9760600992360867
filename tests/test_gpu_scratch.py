"""Whole calls reuse the scratch that a geometry keeps between them, and the
requests of one call share an allocation: from several threads and streams at
once every call gives, bit for bit, what it gives alone, also after calls that
left larger or smaller blocks, and a bad request fails the call that it is in
with its own error, whatever its place."""
import threading

import numpy as np
import pytest

from tests.test_gpu_boundary import dev, small_2d, small_3d

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pet():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_07886_amd as pet
    pet.lib()
    return pet


def calls(pet, G, w, p):
    f, y, r = dev(w.f0), dev(w.y), dev(w.r)

    def reconstruct():
        x = f.clone()
        pet.reconstruct(G, p, x, y, r, 1)
        return x
    return [lambda: G.forward(f, 1), lambda: G.subset_gradient(p, f, y, r, 0), lambda: G.subset_gradient(p, f, y, r, 2),
            lambda: torch.tensor(G.objective(p, f, y, r)), reconstruct]


@pytest.mark.parametrize("dim", [2, 3])
def test_threads_and_streams_share_a_geometry(pet, dim):
    w, p = small_2d() if dim == 2 else small_3d()
    G = pet.Geometry(w.desc)
    todo = calls(pet, G, w, p)
    torch.cuda.synchronize()
    alone = [c().clone() for c in todo]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for n in range(12):
                i = (n + k) % len(todo)
                out = todo[i]()
                s.synchronize()
                if not torch.equal(out, alone[i]):
                    bad.append((k, n, i))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


@pytest.mark.parametrize("where", [0, 1, 3])
def test_batch_reports_its_first_bad_request(pet, where):
    w, p = small_2d()
    G = pet.Geometry(w.desc)
    f = [dev(w.f0) for _ in range(4)]
    y, r = [dev(w.y) for _ in range(4)], [dev(w.r) for _ in range(4)]
    ps = [dict(p) for _ in range(4)]
    y[where][..., 0, 0] = float("nan")
    if where < 3:
        ps[3] = dict(p, mode="OSEM")            # a later one, refused for its mode
    keep = [x.clone() for x in f]
    with pytest.raises(pet.PetOSError) as e:
        pet.reconstruct_batch([G] * 4, ps, f, y, r, [1] * 4)
    assert "y: 1 entries" in str(e.value)
    assert all(torch.equal(a, b) for a, b in zip(f, keep))
    y[where] = dev(w.y)
    if where < 3:
        with pytest.raises(pet.PetOSError) as e:
            pet.reconstruct_batch([G] * 4, ps, f, y, r, [1] * 4)
        assert "OSEM" in str(e.value)
