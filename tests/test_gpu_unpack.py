"""ftwa_unpack against the packed layout's definition: full matrices of both
spins, conjugates below the diagonal, bitwise (values are only moved)."""
import numpy as np
import pytest

from tests._util import unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,M", [
    (1, 1),                       # a single site
    (6, 3), (63, 31), (64, 32), (65, 33),   # column blocks of 64, trajectory blocks of 32 and 64
    (129, 65), (198, 1), (255, 5),          # ragged last blocks, the largest lattice
])
def test_unpack_matches_layout(N, M, dtype):
    import torch
    import paper_2212_04352_amd as ft
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cdt = np.complex64 if dtype == "f32" else np.complex128
    rng = np.random.default_rng(N * 1000 + M)
    P = N * (N + 1) // 2
    packed = (rng.normal(size=(2, P, M)) + 1j * rng.normal(size=(2, P, M))).astype(cdt)
    i, j = np.triu_indices(N)
    packed[:, i == j] = packed[:, i == j].real
    rho = torch.from_numpy(packed).cuda()
    out = torch.empty((M, 2, N, N), dtype=rho.dtype, device="cuda")
    ft.ftwa_unpack(N, M, dtype, rho, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), unpack(packed, N))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,M", [(2, 8), (24, 7), (65, 8), (65, 9), (198, 2)])
def test_unpack_of_few_trajectories(N, M, dtype):
    """Both sides of the line at 8 trajectories between the block sizes."""
    test_unpack_matches_layout(N, M, dtype)
