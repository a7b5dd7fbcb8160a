"""Six and eight steps in one pass of k2_march: cmlbm2d_step(n) gives the same
bits as n calls of one step, which run k2_step alone.

The planes are the smallest that take the longer passes and hit their edges:
rows of whole and of cut strips, odd rows (one cell per lane), a chunk of rows
shorter than the rows that a pass loses, calls whose last passes are shorter.
Every operation is the same in the same order, so the tolerance is zero.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1905_10182_amd.cmlbm2d import Lattice2D  # noqa: E402

DIMS = [(4096, 1100), (2050, 2100), (3001, 1500), (9000, 700), (64, 70000)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("force", ["uniform", "field"])
@pytest.mark.parametrize("dims", DIMS, ids=[f"{a}x{b}" for a, b in DIMS])
def test_long_passes_equal_single_steps(dims, storage, force):
    nx, ny = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + ny)
    f = (0.8 + 0.4 * torch.rand((9, ny, nx), generator=g, device="cuda", dtype=torch.float64)) / 9
    F = 1e-3 * (torch.rand((2, ny, nx), generator=g, device="cuda", dtype=torch.float64) - 0.5)
    A, B = (Lattice2D(nx, ny, tau=0.7, storage=storage, device="cuda:0") for _ in range(2))
    for lat in (A, B):
        if force == "field":
            lat.set_force("field", field=F)
        else:
            lat.set_force("uniform", [1e-4, -2e-5])
        lat.load_populations(f)
    for n in (6, 8, 10, 21):
        print(f"{storage} {nx}x{ny} {force}: {n} steps", flush=True)
        A.step(n)
        for _ in range(n):
            B.step(1)
        assert A.time == B.time
        assert torch.equal(A.populations(), B.populations()), n
