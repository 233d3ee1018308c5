"""The autotuner on small lattices: where a pack of the shared-pack kernel is
the automatic choice, tuning never replaces it by a smaller pack; what it
returns can be forced and gives the automatic plan's results, and automatic
runs after tuning are as fast as before."""
import pytest

pytestmark = pytest.mark.gpu

FIRST_SHARED = 38


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


def _interaction(lat):
    import torch
    i = torch.arange(lat.N, dtype=torch.float64, device="cuda")
    return 3.0 / (1.0 + (i[:, None] - i[None, :]).abs())


def _kernel_ms(ft, prob):
    ms = []
    for _ in range(5):
        timing = ft.new_timing()
        ft.evolve(prob, 1e-3, 40, 40, timing=timing)
        ms.append(timing["ms"].value)
    return min(ms[1:])


# lattices and ensembles whose plan a tuned pack of at most four, or one tuned
# at another ensemble or Hamiltonian, replaced by one of up to 2.7 times its time
@pytest.mark.parametrize("spec,dtype,tuned_at,M,interaction", [
    (("hex", 2, 0), "f32", 4000, 64, False), (("torus", 3, 9), "f64", 64, 64, True),
    (("torus", 6, 6), "f32", 4000, 4000, True), (("armchair", 2, 5), "f64", 64, 20000, True),
])
def test_tuning_keeps_the_packs(ft, spec, dtype, tuned_at, M, interaction):
    import torch
    lat = ft.Lattice(*spec)

    def problem(M, interaction):
        p = ft.Problem.allocate(lat, 3.0, M, lat.fock_start("neel"), dtype)
        if interaction:
            p.u_mat = _interaction(lat)
        ft.sample(p, 4)
        return p
    before = _kernel_ms(ft, problem(M, interaction))
    config = ft.autotune(problem(tuned_at, False))[0]
    after = _kernel_ms(ft, problem(M, interaction))
    print(f"{lat.N} sites {dtype}: configuration {config}, {before:.3f} and {after:.3f} ms",
          flush=True)
    assert config >= FIRST_SHARED
    assert after < 1.25 * before
    a, b = problem(tuned_at, False), problem(tuned_at, False)
    ft.evolve(a, 0.01, 6, 3)
    ft.evolve(b, 0.01, 6, 3, path="resident", config=config)
    assert torch.equal(a.rho, b.rho)
