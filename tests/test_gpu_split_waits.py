"""The split kernel's other ways: the exchange between workgroups that do not
share an XCD's L2 (forced by the host) gives bitwise the results of the one
that stops there, and a bounded wait whose partners are absent gives up, every
workgroup exits, the state stays as it was and the run reports FTWA_ETIMEOUT;
the next run on the same workspace is unaffected."""
import pytest

pytestmark = pytest.mark.gpu

DROP_PARTNERS, FAR_EXCHANGE = 1, 2
FTWA_ETIMEOUT = -6


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


def _pair(ft, lat, M, **kw):
    a, b = (ft.Problem.allocate(lat, 3.3, M, lat.fock_start("neel"), "f64", **kw)
            for _ in range(2))
    ft.sample(a, 6)
    b.rho.copy_(a.rho)
    return a, b


def _variant(prob, lat, variant, steps):
    import torch
    if variant == "potential":
        prob.v_site = torch.linspace(-1, 1, lat.N, dtype=torch.float64, device="cuda")
        prob.v_env = torch.linspace(0, 1, 2 * steps + 1, dtype=torch.float64, device="cuda")
    elif variant == "interaction":
        i = torch.arange(lat.N, dtype=torch.float64, device="cuda")
        prob.u_mat = 3.0 / (1.0 + (i[:, None] - i[None, :]).abs())
    elif variant == "hopping":
        prob.hop_w = torch.ones((2 * steps + 1, lat.N, 3), dtype=torch.complex128, device="cuda")


@pytest.mark.parametrize("spec,config,M", [
    (("hex", 5, 0), 19, 70), (("armchair", 10, 20), 20, 45), (("armchair", 10, 20), 21, 5),
    (("hex", 5, 0), 22, 9), (("armchair", 8, 14), 37, 9), (("hex", 2, 0), 37, 83),
])
def test_exchange_across_xcds(ft, spec, config, M):
    import torch
    lat, steps = ft.Lattice(*spec), 6
    for variant in ("plain", "potential", "interaction", "hopping"):
        print(f"{lat.N} sites, configuration {config}, {variant}", flush=True)
        near, far = _pair(ft, lat, M)
        for p in (near, far):
            _variant(p, lat, variant, steps)
        ft.evolve(near, 0.02, steps, 3, path="resident", config=config)
        ft.evolve(far, 0.02, steps, 3, path="resident", config=config, drop_partners=FAR_EXCHANGE)
        for name in ("rho", "S1", "S2"):
            assert torch.equal(getattr(near, name), getattr(far, name))


@pytest.mark.parametrize("spec,config", [(("hex", 5, 0), 19), (("armchair", 10, 20), 20),
                                         (("armchair", 10, 20), 21), (("hex", 5, 0), 22),
                                         (("armchair", 8, 14), 37), (("hex", 5, 0), -1)])
def test_absent_partners_time_out(ft, spec, config):
    """config -1: with invariant monitors, where the run is a launch per record
    interval and the launches after the first have nothing to wait for."""
    import torch
    lat, steps, every = ft.Lattice(*spec), 6, 2
    kw = dict(path="resident", config=config) if config >= 0 else {}
    p, q = _pair(ft, lat, 20, track_invariants=config < 0)
    start = p.rho.clone()
    with pytest.raises(ft.FtwaError) as e:
        ft.evolve(p, 0.02, steps, every, spin_limit=200, drop_partners=DROP_PARTNERS, **kw)
    assert e.value.status == FTWA_ETIMEOUT
    torch.cuda.synchronize()
    assert torch.equal(p.rho, start)
    ft.evolve(p, 0.02, steps, every, **kw)
    ft.evolve(q, 0.02, steps, every, path="stream")
    assert torch.equal(p.rho, q.rho)
