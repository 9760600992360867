"""The server's device-memory budget: a request is charged what it allocates, in
3D with the projectors' own layout of the subset sinogram; one that fits the
whole budget only bin by bin is taken and charged for that; and the geometry
that a request is about to use is not evicted for it.  (Simulated executor; the
device runs the tight budget too.)"""
import time

import numpy as np
import pytest

from synth import configs


@pytest.fixture(scope="module")
def pet():
    import os
    import paper_2111_07886_amd as pet
    if not os.path.exists(pet.LIB_PATH):
        from paper_2111_07886_amd import build
        build.build()
    return pet


def desc(n=48, nz=12, rd=10, M=2):
    nr = 2 * int(np.ceil(n / np.sqrt(2))) + 3
    return configs.desc_3d(n, nz, 16 * M, nr, 300.0 / n, 3.0, nz, rd, M)


def floats(d, quads):
    """Floats of a P2 request's scratch: the subset sinogram, five images (G, mu,
    nu, the z-fastest copy, the penalty gradient) and nothing else of size."""
    planes = d["n_rings"] + sum(2 * (d["n_rings"] - k) for k in range(1, d["max_ring_diff"] + 1))
    sub = -(-d["n_angles"] // d["n_subsets"])
    q = 4 * sub * (d["max_ring_diff"] + 1) * ((d["n_radial"] + 1) // 2) * d["nz"]
    return (q if quads else sub * planes * d["n_radial"]) + 5 * d["nx"] * d["ny"] * d["nz"]


def charged(pet, d, p):
    """(bytes in use while the request runs, after it: its geometry's)"""
    S = pet.Server(1 << 40, 4, simulate=True, step_us=2000)
    t = S.submit(d, p, n_iter=2)
    while S.stats()["active"] == 0:
        time.sleep(0.001)
    per = S.stats()["bytes_in_use"]
    S.wait(t)
    geo = S.stats()["bytes_in_use"]
    S.close()
    return per, geo


def test_quads_are_counted(pet):
    d, p = desc(), configs.params_3d()
    assert floats(d, True) > 1.3 * floats(d, False)
    per, geo = charged(pet, d, p)
    assert 4 * floats(d, True) <= per - geo <= 1.1 * 4 * floats(d, True) + 65536


def test_a_tight_budget_takes_the_request_bin_by_bin(pet):
    d, p = desc(), configs.params_3d()
    per, geo = charged(pet, d, p)
    budget = geo + (4 * floats(d, False) + per - geo) // 2      # between the two layouts
    S = pet.Server(budget, 4, simulate=True, step_us=2000)
    ts = [S.submit(d, p, n_iter=2) for _ in range(3)]
    most = 0
    while S.stats()["active"] + S.stats()["queued"] > 0:
        most = max(most, S.stats()["bytes_in_use"])
        time.sleep(0.0005)
    assert all(S.wait(t)["status"] == 0 for t in ts)
    assert geo < most <= budget and S.stats()["max_active"] == 1
    S.close()


def test_its_own_geometry_is_not_evicted(pet):
    """A longer request of the only cached geometry, when memory is short: that
    geometry stays (it had been looked up before the eviction)."""
    d, p = desc(), configs.params_3d()
    per, geo = charged(pet, d, p)
    S = pet.Server(per + 4096, 4, simulate=True, step_us=10)
    for n in (2, 1000, 2):                  # (the long schedule is 16 KB more)
        assert S.wait(S.submit(d, p, n_iter=n))["status"] == 0
        assert S.stats()["geometries_cached"] == 1 and S.stats()["bytes_in_use"] == geo
    S.close()


@pytest.mark.gpu
def test_tight_budget_on_the_device(pet):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from synth import phantoms
    from tests.test_gpu_boundary import dev
    d = desc()
    w = phantoms.make_3d(d, seed=5, n_ell=3, counts=1e6, bg_uniform=0.1, bg_scatter=0.1, scatter_sigma_bins=4.0)
    p = dict(configs.params_3d(U=w.U), lambda0=0.01)
    per, geo = charged(pet, d, p)
    y, r, want = dev(w.y), dev(w.r), dev(w.f0)
    pet.reconstruct(pet.Geometry(d), p, want, y, r, 2)
    torch.cuda.synchronize()
    for budget, exact in ((1 << 32, True), (geo + (4 * floats(d, False) + per - geo) // 2, False)):
        f = dev(w.f0)
        torch.cuda.synchronize()
        S = pet.Server(budget, 2)
        res = [S.wait(t) for t in [S.submit(d, p, f, y, r, 2, want_objective=True)]]
        S.close()
        print(f"[server-budget] {budget}: {res[0]['status']} {res[0]['message']}", flush=True)
        assert res[0]["status"] == 0
        assert torch.equal(f, want) == exact
        assert float((f - want).norm() / want.norm()) <= 1e-5
