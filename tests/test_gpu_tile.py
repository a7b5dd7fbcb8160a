"""Several steps of a small lattice in one launch (k_tile): cmlbm_step(n) gives
the same bits as n calls of one step, which go through k_step alone.

Lattices at the edges of the path: one tile per axis with a halo that meets
itself around the period, tiles cut in each axis, the most tiles that FP64
takes by threes, the most that it takes by twos, batches.  Calls of 2 to 5
steps cover passes of three, of two and the step left over.  The reference is
the one-step kernel on the same state, itself checked against the oracle; every
cell update is the same operations in the same order, so the tolerance is zero.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import workloads as W  # noqa: E402
from paper_1905_10182_amd import Lattice  # noqa: E402

DIMS = {
    "one_tile_rows": (8, 8, 8, 1),
    "cut_tiles": (9, 11, 13, 2),
    "narrow_batch": (8, 9, 8, 30),
    "fp64_threes_limit": (32, 32, 16, 1),
    "fp64_twos_limit": (32, 32, 32, 1),
}


@pytest.mark.parametrize("dims", list(DIMS.values()), ids=list(DIMS))
@pytest.mark.parametrize("storage", ["fp32", "fp64"])
@pytest.mark.parametrize("wall,solid,field", [((0, 0, 0), False, False), ((0, 0, 0), False, True),
                                              ((0, 1, 0), True, False), ((1, 1, 1), True, True)],
                         ids=["periodic", "field", "wall", "box_field"])
def test_same_bits_as_single_steps(dims, storage, wall, solid, field):
    nx, ny, nz, nb = dims
    print("tile", dims, storage, wall, solid, field, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)

    def rand(*shape):
        return torch.rand(shape, generator=gen, device="cuda", dtype=torch.float64)

    shape = (nb, nz, ny, nx)
    f = (0.8 + 0.4 * rand(27, *shape)) / 27
    F = 1e-3 * (rand(3, *shape) - 0.5)
    S = rand(*shape) < 0.1
    a, b = (Lattice(nx, ny, nz, nbatch=nb, tau=0.7, storage=storage, wall=wall, solid=solid, device="cuda:0")
            for _ in range(2))
    for lat in (a, b):
        if solid:
            lat.set_solid(S)
        if field:
            lat.set_force("field", field=F)
        else:
            lat.set_force("batch", W.generator(3).uniform(-1e-4, 1e-4, size=(nb, 3)))
        lat.load_populations(f)
    for n in (2, 3, 4, 5):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert np.array_equal(a.populations().cpu().numpy(), b.populations().cpu().numpy()), n
        assert a.time == b.time
