"""Invariant monitors on the split resident kernel, which is launched once per
record interval with the invariant sums of the stored state in between:
bitwise the stream kernels' states and monitors, with and without a
potential, ragged last intervals, single-step intervals, no steps, trajectory
windows and as a graph."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


def _problem(ft, lat, M, variant, steps, rho):
    import torch
    prob = ft.Problem.allocate(lat, 3.3, M,
                               lat.fock_start("neel"), "f64", track_invariants=True)
    if rho is None:
        ft.sample(prob, 8)
    else:
        prob.rho.copy_(rho)
    rng = np.random.default_rng(4)
    tau = np.arange(2 * steps + 1) * 0.01
    if variant == "potential":
        prob.v_site = torch.from_numpy(rng.uniform(-1, 1, lat.N)).cuda()
        prob.v_env = torch.from_numpy(np.exp(-((tau - 0.05) / 0.03) ** 2)).cuda()
    return prob


@pytest.mark.parametrize("variant", ["plain", "potential"])
@pytest.mark.parametrize("M,steps,every,chunk", [(37, 11, 4, 0), (9, 3, 1, 4), (5, 2, 8, 0),
                                                 (6, 0, 1, 0)])
def test_monitored_split_runs_match_the_stream_path(ft, variant, M, steps, every, chunk):
    import torch
    lat = ft.Lattice("hex", 5, 0)
    print(f"{variant} {M} trajectories {steps} steps every {every} chunk {chunk}", flush=True)
    a = _problem(ft, lat, M, variant, steps, None)
    start = a.rho.clone()
    b = _problem(ft, lat, M, variant, steps, start)
    c = _problem(ft, lat, M, variant, steps, start)
    ft.evolve(a, 0.02, steps, every, path="stream", traj_chunk=chunk)
    ft.evolve(b, 0.02, steps, every, traj_chunk=chunk)
    graph = ft.EvolveGraph(c, 0.02, steps, every, traj_chunk=chunk)
    for _ in range(3):
        c.rho.copy_(start)
        graph.launch()
        graph.check()
        torch.cuda.synchronize()
        for x in (b, c):
            assert torch.equal(a.rho, x.rho)
            assert torch.equal(a.inv, x.inv)
            assert torch.allclose(a.S1, x.S1, rtol=1e-12, atol=1e-12)
            assert torch.allclose(a.S2, x.S2, rtol=1e-12, atol=1e-12)
