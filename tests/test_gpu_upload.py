"""ftwa_lattice_upload: every table of a lattice in one allocation that
ftwa_free_lattice gives back, also where several threads upload one lattice at
once; runs on it equal those on a lattice uploaded alone."""
import threading

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


def test_upload_gives_its_memory_back(ft):
    import torch

    def cycle():
        for spec in (("armchair", 2, 5), ("torus", 3, 9), ("hex", 4, 0), ("armchair", 10, 20)):
            lat = ft.Lattice(*spec)
            lat.upload()
            lat.upload()
            lat.close()
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]
    cycle()
    assert cycle() == cycle()


@pytest.mark.parametrize("spec", [("torus", 2, 3), ("torus", 3, 9), ("hex", 5, 0)])
def test_threads_upload_one_lattice(ft, spec):
    import torch
    torch.cuda.init()
    one, many = ft.Lattice(*spec), ft.Lattice(*spec)
    one.upload()
    errors = []

    def upload():
        try:
            many.upload()
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(e)
    threads = [threading.Thread(target=upload) for _ in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for dtype in ("f64", "f32"):
        a, b = (ft.Problem.allocate(lat, 2.0, 33, lat.fock_start("neel"), dtype)
                for lat in (one, many))
        for p in (a, b):
            ft.sample(p, 2)
            ft.evolve(p, 0.02, 6, 3)
        assert torch.equal(a.rho, b.rho) and torch.equal(a.S2, b.S2)
