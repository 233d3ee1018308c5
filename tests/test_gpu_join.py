"""Runs of many instances whose plans depend on each other: lattices of
different sizes that share one launch in the largest one's shape (few
trajectories each), and scans on one lattice whose trajectories count
together; bitwise the states of one run per instance, moments to 1e-12, as
plain runs, in several passes and as a graph."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [("hex", 4, 0), ("armchair", 2, 5), ("torus", 2, 3), ("hex", 2, 0), ("torus", 3, 9),
         ("torus", 6, 6)]
STEPS, EVERY = 8, 4


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


def _problem(ft, lat, U, M, dtype, variant, k):
    import torch
    p = ft.Problem.allocate(lat, U, M, lat.fock_start("neel"), dtype)
    rng = np.random.default_rng(k)
    if variant == "potential":
        p.v_site = torch.from_numpy(rng.uniform(-1, 1, lat.N)).cuda()
        p.v_env = torch.linspace(0, 1, 2 * STEPS + 1, dtype=torch.float64, device="cuda")
    elif variant == "interaction":
        x = rng.uniform(-0.2, 0.2, (lat.N, lat.N))
        p.u_mat = torch.from_numpy(3.3 * np.eye(lat.N) + x + x.T).cuda()
    elif variant == "hopping":
        w = np.exp(1j * rng.uniform(0, 1, (2 * STEPS + 1, lat.N, 3)))
        p.hop_w = torch.from_numpy(w).cuda()
    ft.sample(p, 3 + k)
    return p


def _check(ft, make, chunk=0):
    import torch
    together, single = make(), make()
    starts = [p.rho.clone() for p in together]
    for q in single:
        ft.evolve(q, 0.02, STEPS, EVERY)
    ft.evolve(together, 0.02, STEPS, EVERY, traj_chunk=chunk)

    def same():
        for p, q in zip(together, single):
            assert torch.equal(p.rho, q.rho)
            assert torch.allclose(p.S1, q.S1, rtol=1e-12, atol=1e-12)
            assert torch.allclose(p.S2, q.S2, rtol=1e-12, atol=1e-12)
    same()
    graph = ft.EvolveGraph(together, 0.02, STEPS, EVERY, traj_chunk=chunk)
    for _ in range(2):
        for p, s in zip(together, starts):
            p.rho.copy_(s)
        torch.cuda.synchronize()
        graph.launch()
        graph.check()
        same()


@pytest.mark.parametrize("variant", ["plain", "potential", "interaction", "hopping"])
@pytest.mark.parametrize("M,chunk", [(5, 0), (45, 0), (9, 4)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_lattices_of_different_sizes(ft, dtype, M, chunk, variant):
    lats = [ft.Lattice(*s) for s in SIZES[2 if dtype == "f64" or variant == "hopping" else 0:]]
    print(f"{dtype} {variant} {M} trajectories", flush=True)
    _check(ft, lambda: [_problem(ft, lat, 1.0 + 0.3 * k, M + k % 2, dtype, variant, k)
                        for k, lat in enumerate(lats)], chunk)


@pytest.mark.parametrize("variant", ["plain", "interaction"])
@pytest.mark.parametrize("spec,count,M", [(("armchair", 2, 5), 24, 160), (("torus", 3, 9), 12, 70)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_scans_on_one_lattice(ft, dtype, spec, count, M, variant):
    lat = ft.Lattice(*spec)
    print(f"{dtype} {variant} {lat.N} sites {count} x {M} trajectories", flush=True)
    _check(ft, lambda: [_problem(ft, lat, 0.5 * k, M, dtype, variant, 7) for k in range(count)])
