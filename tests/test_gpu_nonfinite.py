"""States that have blown up, through the kernels that take several steps in one
launch: NaN, infinities and cells of zero density spread exactly as through
single steps (k_tile, k2_tile, k2_march; k_march's own test counts the cells).

The populations after a call of n steps and after n calls of one step are the
same: not-a-number at the same places, every other value equal.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1905_10182_amd import Lattice  # noqa: E402
from paper_1905_10182_amd.cmlbm2d import Lattice2D  # noqa: E402


def blown_up(q, shape, seed):
    """Random populations with a NaN, both infinities and an empty cell, in cells apart."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    f = (0.8 + 0.4 * torch.rand((q,) + shape, generator=g, device="cuda", dtype=torch.float64)) / q
    flat = f.view(q, -1)
    cells = torch.randperm(flat.shape[1], generator=g, device="cuda")[:4]
    flat[1, cells[0]] = float("nan")
    flat[2, cells[1]] = float("inf")
    flat[3, cells[2]] = float("-inf")
    flat[:, cells[3]] = 0.0
    return f


def check(make, q, shape, n):
    lats = []
    for _ in range(2):
        lat = make()
        lat.load_populations(blown_up(q, shape, 4))
        lats.append(lat)
    A, B = lats
    A.step(n)
    for _ in range(n):
        B.step(1)
    a, b = A.populations(), B.populations()
    bad = torch.isnan(a)
    assert bad.any() and not bad.all()
    assert torch.equal(bad, torch.isnan(b))
    assert torch.equal(a[~bad], b[~bad])


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("wall", [(0, 0, 0), (0, 1, 0)])
@pytest.mark.parametrize("dims,n", [((32, 24, 16), 3), ((32, 24, 16), 2)], ids=["three", "two"])
def test_small_lattices(dims, n, wall, storage):
    nx, ny, nz = dims
    print("nonfinite", dims, n, wall, storage, flush=True)
    check(lambda: Lattice(nx, ny, nz, tau=0.7, storage=storage, wall=wall, device="cuda:0"), 27, (1, nz, ny, nx), n)


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("dims,n", [((300, 211), 7), ((1025, 1100), 4), ((4096, 1100), 6), ((8192, 1750), 8)],
                         ids=["tile", "march4", "march6", "march8"])
def test_planes(dims, n, storage):
    nx, ny = dims
    print("nonfinite", dims, n, storage, flush=True)
    check(lambda: Lattice2D(nx, ny, tau=0.7, storage=storage, device="cuda:0"), 9, (ny, nx), n)
