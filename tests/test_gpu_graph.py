"""Calls of an even number of steps captured into a HIP graph: every replay
advances the state by that many steps.

The graph is replayed several times with the program's own work between, and
the state after each replay is compared with a lattice that takes the steps by
ordinary calls, bit for bit.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1905_10182_amd import Lattice  # noqa: E402


def check_replays(make, f, n):
    lats = []
    for _ in range(2):
        lat = make()
        lat.load_populations(f)
        lat.step(n)  # an ordinary call first
        lats.append(lat)
    A, B = lats
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.step(n)
    for replay in range(3):
        graph.replay()
        B.step(n)
        pops = A.populations()  # reads the state between replays
        torch.cuda.synchronize()
        assert torch.equal(pops, B.populations()), replay
    A.step(n)  # and ordinary calls go on from there
    B.step(n)
    assert torch.equal(A.populations(), B.populations())
    # the same lattice by turns: a new state, ordinary calls, the new state again, the graph
    f2 = f.flip(-1).contiguous()
    A.load_populations(f2)
    A.step(n)
    A.step(2)
    want = A.populations()
    A.load_populations(f2)
    graph.replay()
    A.step(2)
    assert torch.equal(A.populations(), want)


def populations(q, shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    return (0.8 + 0.4 * torch.rand((q,) + shape, generator=g, device="cuda", dtype=torch.float64)) / q


# two-step launches alone, with three-step ones, paired; single steps; the path through the nine numbers
@pytest.mark.parametrize("dims,wall", [((8, 8, 8), (0, 0, 0)), ((8, 60, 60), (0, 1, 0)), ((32, 32, 32), (0, 1, 0)),
                                       ((96, 96, 96), (0, 0, 0))])
@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [2, 4, 6])
def test_replays_advance_the_state(dims, wall, storage, n):
    nx, ny, nz = dims
    print("graph", dims, storage, n, flush=True)
    check_replays(lambda: Lattice(nx, ny, nz, tau=0.7, storage=storage, wall=wall, device="cuda:0"),
                  populations(27, (1, nz, ny, nx)), n)


@pytest.mark.parametrize("dims", [(64, 64), (300, 211), (1025, 1100)])
@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [2, 6, 8, 10])
def test_replays_advance_the_plane_state(dims, storage, n):
    from paper_1905_10182_amd.cmlbm2d import Lattice2D
    nx, ny = dims
    print("graph", dims, storage, n, flush=True)
    check_replays(lambda: Lattice2D(nx, ny, tau=0.7, storage=storage, device="cuda:0"), populations(9, (ny, nx)), n)
