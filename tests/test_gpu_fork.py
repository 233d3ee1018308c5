"""Graphs of batches whose groups run side by side: every replay, with the
program's own work between the replays, equals the runs one by one, states
bitwise and moments to 1e-12; with and without a group whose workgroups wait
for each other, and with several passes over the trajectories."""
import pytest

pytestmark = pytest.mark.gpu

SMALL = [("armchair", 2, 5), ("torus", 2, 3), ("hex", 2, 0), ("torus", 3, 9), ("hex", 4, 0)]


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("extra,M,chunk", [((), 33, 0), ((("hex", 5, 0),), 20, 0), ((), 33, 16)],
                         ids=["small", "with-split", "passes"])
def test_side_by_side_groups(ft, dtype, extra, M, chunk):
    import torch
    steps, every = 12, 4
    lats = [ft.Lattice(*s) for s in SMALL + list(extra)]
    problems, starts, single = [], [], []
    for k, lat in enumerate(lats):
        p = ft.Problem.allocate(lat, 1.0 + 0.5 * k, M, lat.fock_start("neel"), dtype)
        ft.sample(p, 3 + k)
        problems.append(p)
        starts.append(p.rho.clone())
        q = ft.Problem.allocate(lat, 1.0 + 0.5 * k, M, lat.fock_start("neel"), dtype)
        q.rho.copy_(p.rho)
        ft.evolve(q, 0.02, steps, every)
        single.append(q)
    graph = ft.EvolveGraph(problems, 0.02, steps, every, traj_chunk=chunk)
    for _ in range(3):
        for p, s in zip(problems, starts):
            p.rho.copy_(s)
            p.S1.fill_(7.0)
            p.S2.fill_(7.0)
        torch.cuda.synchronize()
        graph.launch()
        graph.check()
        for p, q in zip(problems, single):
            assert torch.equal(p.rho, q.rho)
            assert torch.allclose(p.S1, q.S1, rtol=1e-12, atol=1e-12)
            assert torch.allclose(p.S2, q.S2, rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_groups_with_shared_moments_keep_their_order(ft, dtype):
    """Two instances of different groups (one with a potential) whose moments
    meet in one S1 and S2: every replay gives the sum of both runs."""
    import torch
    lat, M, steps, every = ft.Lattice("torus", 2, 3), 40, 8, 4
    potential = {"v_site": torch.linspace(-1, 1, lat.N, dtype=torch.float64, device="cuda"),
                 "v_env": torch.ones(2 * steps + 1, dtype=torch.float64, device="cuda")}

    def problems():
        out = [ft.Problem.allocate(lat, 2.0, M, lat.fock_start("neel"), dtype, traj_offset=k * M)
               for k in range(2)]
        for name, value in potential.items():
            setattr(out[1], name, value)
        ft.sample(out, 5)
        return out

    single, pair = problems(), problems()
    for q in single:
        ft.evolve(q, 0.02, steps, every)
    S1, S2 = (sum(getattr(q, name) for q in single) for name in ("S1", "S2"))
    starts = [p.rho.clone() for p in pair]
    pair[0].ensure_moments(steps // every + 1)
    pair[1].S1, pair[1].S2 = pair[0].S1, pair[0].S2
    graph = ft.EvolveGraph(pair, 0.02, steps, every)
    for _ in range(5):
        for p, s in zip(pair, starts):
            p.rho.copy_(s)
        torch.cuda.synchronize()
        graph.launch()
        graph.check()
        for p, q in zip(pair, single):
            assert torch.equal(p.rho, q.rho)
        assert torch.allclose(pair[0].S1, S1, rtol=1e-12, atol=1e-12)
        assert torch.allclose(pair[0].S2, S2, rtol=1e-12, atol=1e-12)
