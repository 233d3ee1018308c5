"""The split kernel's halo exchange at its edges, bitwise against the oracle:
a lattice whose halo takes more than one round of reads per thread, one whose
import table does not fit in LDS, the smallest parts, and several trajectories
in turn through every group."""
import numpy as np
import pytest

from tests._util import pack, unpack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


@pytest.mark.parametrize("kind,a,b,config,M,variant", [
    ("torus", 5, 13, 19, 3, "plain"),       # 130 sites, two parts: more than 512 entries per class
    ("armchair", 8, 25, 20, 2, "hopping"),  # 200 sites: no room for the import table in LDS
    ("armchair", 8, 14, 37, 5, "plain"),    # 110 sites: two parts of (4, 4) slots
    ("hex", 2, 0, 37, 83, "potential"),     # 24 sites, more trajectories than groups
    ("hex", 1, 0, 21, 45, "potential"),     # 6 sites in 4 parts
])
def test_halo_exchange(ft, orc, kind, a, b, config, M, variant):
    import torch
    dt, steps, every = 0.01, 5, 2
    olat, lat = orc.Lattice(kind, a, b), ft.Lattice(kind, a, b)
    print(f"{kind} {a}x{b} {lat.N} sites, configuration {config}", flush=True)
    n0 = orc.fock_start(olat, "random", 2)
    rho0 = orc.sample(olat, n0, 2, M)
    prob = ft.Problem.allocate(lat, 3.3, M, n0, "f64")
    prob.rho.copy_(torch.from_numpy(pack(rho0)))
    kw = {}
    rng = np.random.default_rng(2)
    tau = np.arange(2 * steps + 1) * dt / 2
    if variant == "potential":
        v, env = rng.uniform(-1, 1, lat.N), np.cos(3.0 * tau)
        prob.v_site, prob.v_env = torch.from_numpy(v).cuda(), torch.from_numpy(env).cuda()
        kw = dict(vsite=v, env=env)
    elif variant == "hopping":
        x = rng.uniform(0, 1, lat.N)

        def table(nbr, deg, fill):
            w = np.full((tau.size, lat.N, 3), fill, dtype=np.complex128)
            for i in range(lat.N):
                for n in range(int(deg[i])):
                    w[:, i, n] = np.exp(1j * np.sin(30 * tau) * (x[i] - x[int(nbr[i][n])]))
            return w
        prob.hop_w = torch.from_numpy(table(lat.nbr, lat.deg, np.nan)).cuda()
        kw = dict(hop=table(olat.nbr, olat.deg, 0.0))
    ft.evolve(prob, dt, steps, every, path="resident", config=config)
    y_ref, X_ref, _ = orc.evolve(olat, 3.3, rho0, dt, steps, every, **kw)
    torch.cuda.synchronize()
    got = unpack(prob.rho.cpu().numpy(), lat.N)
    assert np.array_equal(got, y_ref), np.max(np.abs(got - y_ref))
    S1r, S2r = orc.moments(X_ref)
    assert np.allclose(prob.S1.cpu().numpy(), S1r, rtol=1e-12, atol=1e-12)
    assert np.allclose(prob.S2.cpu().numpy(), S2r, rtol=1e-12, atol=1e-12)
