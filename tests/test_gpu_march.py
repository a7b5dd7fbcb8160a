"""The moment path of a multi-step call (k_march): cmlbm_step(n) gives the same
bits as n calls of one step, which go through k_step alone.

The lattices are the smallest that take the path (some tens of thousands of
wavefronts; smaller ones stay with k_step) and hit its edges: tiles cut in x
and y, a tile that is a whole periodic row, rows of a few cells, a last chunk
of planes that is shorter, the halo of a batch member's first and last plane,
the 6- and the 12-row tile.  The reference is the solver's own one-step kernel
on the same state, itself checked against the oracle; every operation of the
two paths is the same in the same order, so the tolerance is zero.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import workloads as W  # noqa: E402
from paper_1905_10182_amd import Lattice  # noqa: E402

DIMS = {
    "whole_rows": (64, 32, 32, 16),
    "cut_tiles": (250, 50, 41, 2),
    "narrow_rows": (5, 11, 40, 512),
    "one_column_over": (65, 30, 62, 14),
}


def pair(dims, storage, wall, solid, field, seed=5):
    """Two lattices in the same state: a random non-equilibrium one, with a
    random per-cell force or a per-member one, and random solid cells."""
    nx, ny, nz, nb = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def rand(*shape):
        return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)

    shape = (nb, nz, ny, nx)
    f = (0.8 + 0.4 * rand(27, *shape)) / 27
    F = 1e-3 * (rand(3, *shape) - 0.5)
    S = rand(*shape) < 0.1
    out = []
    for _ in range(2):
        lat = Lattice(nx, ny, nz, nbatch=nb, tau=0.7, storage=storage, wall=wall, solid=solid, device="cuda:0")
        if solid:
            lat.set_solid(S)
        if field:
            lat.set_force("field", field=F)
        else:
            lat.set_force("batch", W.generator(seed).uniform(-1e-4, 1e-4, size=(nb, 3)))
        lat.load_populations(f)
        out.append(lat)
    return out


@pytest.mark.parametrize("dims", list(DIMS.values()), ids=list(DIMS))
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("wall,solid,field", [((0, 0, 0), False, False), ((0, 0, 0), False, True),
                                              ((0, 1, 0), True, False), ((1, 1, 1), True, True)],
                         ids=["periodic", "periodic_field", "spheres", "closed_field"])
def test_steps_of_one_call_equal_single_steps(dims, storage, wall, solid, field):
    A, B = pair(dims, storage, wall, solid, field)
    for n in (2, 3, 6):
        print(f"{storage} {dims} walls {wall} solid {solid} field {field}: {n} steps", flush=True)
        A.step(n)
        for _ in range(n):
            B.step(1)
        assert A.time == B.time
        assert torch.equal(A.populations(), B.populations()), n
    A.close()
    B.close()


def test_restart_inside_a_run_is_bitwise():
    """12 steps in one call equal 5, a checkpoint restored into a fresh handle, and 7."""
    wl = W.taylor_green(128, re=400.0)
    lats = []
    for _ in range(2):
        lat = Lattice(128, 128, 128, tau=wl["tau"], storage="fp32", device="cuda:0")
        lat.init(wl["rho"], wl["u"])
        lats.append(lat)
    lats[0].step(12)
    lats[1].step(5)
    blob, t = lats[1].save_state()
    C = Lattice(128, 128, 128, tau=wl["tau"], storage="fp32", device="cuda:0")
    C.restore_state(blob, t)
    C.step(7)
    assert C.time == 12 and torch.equal(lats[0].populations(), C.populations())


def test_blow_up_is_reported_after_a_call_of_many_steps():
    """A non-finite cell spreads through the moment path and is counted."""
    from paper_1905_10182_amd.cmlbm import EUNSTABLE, RED, CmlbmError
    lat = Lattice(64, 64, 64, nbatch=4, tau=0.7, storage="fp32", device="cuda:0")
    u = np.zeros((3, 4, 64, 64, 64))
    u[0, 2, 10, 11, 12] = np.nan
    lat.init(None, u)
    lat.step(4)
    r = lat.reduce(allow_unstable=True)
    assert list(r[:, RED["nonfinite"]] > 0) == [False, False, True, False]
    with pytest.raises(CmlbmError) as e:
        lat.reduce()
    assert e.value.code == EUNSTABLE
