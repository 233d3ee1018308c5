"""The packs of whole trajectories on small lattices (the shared-pack resident
kernels) through the C ABI: every shape forced on graphs with missing
neighbours, and the automatic choice on both sides of its site, ensemble and
variant rules, bitwise equal to the oracle (small ensembles) and to the stream
kernels (ensembles that fill the chip, a ragged last pack); moments to 1e-12.
"""
import numpy as np
import pytest

from tests._util import pack, unpack

pytestmark = pytest.mark.gpu

FIRST_SHARED = 38  # six FP64 shapes, then six FP32 shapes
DT, STEPS, EVERY = 0.01, 6, 3


@pytest.fixture(scope="module")
def ft():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2212_04352_amd as ft
    ft.load()
    return ft


def _host(x):
    import torch
    torch.cuda.synchronize()
    return x.detach().cpu().numpy()


def _chain(n):
    return ("custom", n, [(k, k + 1) for k in range(n - 1)], [k % 2 for k in range(n)])


# a comb with one isolated site: degrees 0..3, sublattices of 5 and 4 sites
COMB = ("custom", 9, [(0, 1), (1, 2), (2, 3), (1, 4), (3, 5), (5, 6), (5, 7)],
        [0, 1, 0, 1, 0, 0, 1, 1, 0])


def _lattices(ft, orc, spec, t):
    if spec[0] == "custom":
        _, n, bonds, sub = spec
        return (ft.Lattice("custom", 0, 0, t, bonds=bonds, sublattice=sub, n_sites=n),
                orc.Lattice.from_bonds(n, bonds, sub, t=t))
    return ft.Lattice(*spec, t), orc.Lattice(*spec, t)


def _variant(variant, lat, olat, seed):
    """The variant's attributes of a Problem and the same as arguments of the oracle."""
    rng = np.random.default_rng(seed)
    N = olat.N
    tau = np.arange(2 * STEPS + 1) * DT / 2
    if variant == "potential":
        v, env = rng.uniform(-1, 1, N), np.exp(-((tau - 0.03) / 0.02) ** 2)
        return {"v_site": v, "v_env": env}, {"vsite": v, "env": env}
    if variant == "interaction":
        x = rng.uniform(-0.2, 0.2, (N, N))
        u = 3.3 * np.eye(N) + x + x.T
        return {"u_mat": u}, {"umat": u}
    if variant == "hopping":
        x = rng.uniform(0, 1, (N, 2))

        def table(nbr, deg, fill):
            w = np.full((tau.size, N, 3), fill, dtype=np.complex128)
            for i in range(N):
                for k in range(int(deg[i])):
                    d = x[i] - x[int(nbr[i][k])]
                    w[:, i, k] = np.exp(1j * (0.8 * np.sin(30 * tau) * d[0] + 0.4 * tau * d[1]))
            return w
        return ({"hop_w": table(lat.nbr, lat.deg, np.nan)}, {"hop": table(olat.nbr, olat.deg, 0.0)})
    return {}, {}


def _u(attrs):
    return 0.0 if "u_mat" in attrs else 3.3


def _problem(ft, lat, n0, dtype, M, attrs, rho):
    import torch
    prob = ft.Problem.allocate(lat, _u(attrs), M, n0, dtype)
    prob.rho.copy_(rho)
    for name, value in attrs.items():
        setattr(prob, name, torch.from_numpy(np.ascontiguousarray(value)).cuda())
    return prob


def _against_oracle(ft, orc, spec, dtype, variant, M, path, config=-1, t=1.0):
    import torch
    lat, olat = _lattices(ft, orc, spec, t)
    sub = np.asarray(lat.sub, dtype=float)
    n0 = np.array([1.0 - sub, sub])
    rho0 = orc.sample(olat, n0, 5, M)
    cdt = np.complex128 if dtype == "f64" else np.complex64
    attrs, oracle = _variant(variant, lat, olat, 6)
    prob = _problem(ft, lat, n0, dtype, M, attrs, torch.from_numpy(pack(rho0.astype(cdt))))
    ft.evolve(prob, DT, STEPS, EVERY, path=path, config=config)
    y_ref, X_ref, _ = orc.evolve(olat, _u(attrs), rho0, DT, STEPS, EVERY, precision=dtype, **oracle)
    got = unpack(_host(prob.rho), lat.N)
    assert np.array_equal(got, y_ref.astype(cdt)), np.max(np.abs(got - y_ref))
    S1r, S2r = orc.moments(X_ref)
    assert np.allclose(_host(prob.S1), S1r, rtol=1e-12, atol=1e-12)
    assert np.allclose(_host(prob.S2), S2r, rtol=1e-12, atol=1e-12)


VARIANTS = ["plain", "potential", "interaction", "hopping"]


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("shape", range(6))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_every_shape_on_irregular_graphs(ft, orc, dtype, shape, variant):
    config = FIRST_SHARED + shape + (6 if dtype == "f32" else 0)
    if shape == 0 and variant == "interaction":  # one wave has no room for the sums' waves
        with pytest.raises(ft.FtwaError):
            _against_oracle(ft, orc, _chain(7), dtype, variant, 3, "resident", config)
        return
    for spec, M, t in ((_chain(2), 5, 1.0), (_chain(7), 37, 0.7), (COMB, 3, 1.0)):
        print(f"shape {shape} {dtype} {variant} {spec[1]} sites", flush=True)
        _against_oracle(ft, orc, spec, dtype, variant, M, "resident", config, t)


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("spec", [_chain(11), _chain(12), _chain(15), _chain(16), ("hex", 2, 0),
                                  ("torus", 3, 9), ("armchair", 6, 11), ("torus", 6, 6),
                                  ("hex", 4, 0)],
                         ids=lambda s: f"{s[0]}{s[1]}x{s[2]}" if s[0] != "custom" else f"chain{s[1]}")
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_automatic_choice(ft, orc, dtype, spec, variant):
    """Few trajectories against the oracle; an ensemble that fills the chip
    (and one between the rules) against the stream kernels."""
    import torch
    _against_oracle(ft, orc, spec, dtype, variant, 7, "auto")
    lat, olat = _lattices(ft, orc, spec, 1.0)
    sub = np.asarray(lat.sub, dtype=float)
    n0 = np.array([1.0 - sub, sub])
    attrs, _ = _variant(variant, lat, olat, 6)
    for M in (1029, 33003 if lat.N < 17 else 8203 if lat.N < 30 else 3077):
        print(f"{dtype} {variant} {lat.N} sites {M} trajectories", flush=True)
        a = ft.Problem.allocate(lat, 3.3, M, n0, dtype)
        ft.sample(a, 9)
        b = _problem(ft, lat, n0, dtype, M, attrs, a.rho)
        c = _problem(ft, lat, n0, dtype, M, attrs, a.rho)
        ft.evolve(b, DT, STEPS, EVERY)
        ft.evolve(c, DT, STEPS, EVERY, path="stream")
        assert torch.equal(b.rho, c.rho)
        assert torch.allclose(b.S1, c.S1, rtol=1e-12, atol=1e-12)
        assert torch.allclose(b.S2, c.S2, rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("spec", [_chain(3), _chain(13), ("armchair", 2, 7), ("torus", 3, 5)],
                         ids=["chain3", "chain13", "armchair2x7", "torus3x5"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_ensembles_that_end_in_a_partial_round(ft, orc, dtype, spec, variant):
    """Sizes next to the rules' lines; ensembles of a few packs more than run
    at once, so that the last round of every XCD is short or empty."""
    import torch
    lat, olat = _lattices(ft, orc, spec, 1.0)
    sub = np.asarray(lat.sub, dtype=float)
    n0 = np.array([1.0 - sub, sub])
    attrs, _ = _variant(variant, lat, olat, 6)
    for M in (700, 4003):
        print(f"{dtype} {variant} {lat.N} sites {M} trajectories", flush=True)
        a = ft.Problem.allocate(lat, 3.3, M, n0, dtype)
        ft.sample(a, 9)
        b = _problem(ft, lat, n0, dtype, M, attrs, a.rho)
        c = _problem(ft, lat, n0, dtype, M, attrs, a.rho)
        ft.evolve(b, DT, STEPS, EVERY)
        ft.evolve(c, DT, STEPS, EVERY, path="stream")
        assert torch.equal(b.rho, c.rho)
        assert torch.allclose(b.S1, c.S1, rtol=1e-12, atol=1e-12)
        assert torch.allclose(b.S2, c.S2, rtol=1e-12, atol=1e-12)
