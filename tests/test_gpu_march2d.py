"""Several steps in one launch of the D2Q9 solver (k2_tile on small planes,
k2_march on large ones): cmlbm2d_step(n) gives the same bits as n calls of one
step, which run k2_step alone.

The planes hit the edges of both kernels: a row that is exactly a wavefront, one
that is cut into overlapping strips, rows and columns shorter than the strip and
than the rows a launch loses, planes of one cell, odd rows (one cell per lane),
and step counts with every remainder.  The reference is the solver's own
one-step kernel, itself checked against the oracle; every operation is the same
in the same order, so the tolerance is zero.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1905_10182_amd.cmlbm2d import Lattice2D  # noqa: E402

SMALL = [(64, 33), (128, 20), (1, 9), (9, 1), (1, 1), (2, 3), (37, 13), (50, 2), (58, 101), (300, 211)]
LARGE = [(1025, 1100), (2049, 1500), (4096, 900), (6000, 601)]


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("force", ["uniform", "field"])
@pytest.mark.parametrize("dims", SMALL + LARGE, ids=[f"{a}x{b}" for a, b in SMALL + LARGE])
def test_steps_of_one_call_equal_single_steps(dims, storage, force):
    nx, ny = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + 7 * ny)
    f = (0.8 + 0.4 * torch.rand((9, ny, nx), generator=g, device="cuda", dtype=torch.float64)) / 9
    F = 1e-3 * (torch.rand((2, ny, nx), generator=g, device="cuda", dtype=torch.float64) - 0.5)
    lats = []
    for _ in range(2):
        lat = Lattice2D(nx, ny, tau=0.7, storage=storage, device="cuda:0")
        if force == "field":
            lat.set_force("field", field=F)
        else:
            lat.set_force("uniform", [1e-4, -2e-5])
        lat.load_populations(f)
        lats.append(lat)
    A, B = lats
    for n in (2, 3, 4, 7, 12):
        print(f"{storage} {nx}x{ny} {force}: {n} steps", flush=True)
        A.step(n)
        for _ in range(n):
            B.step(1)
        assert A.time == B.time
        assert torch.equal(A.populations(), B.populations()), n
