"""The moment path (k_march) under its blocked workgroup order, and on whole
periodic rows narrower than a tile: cmlbm_step(n) gives the same bits as n calls
of one step.  That these lattices take the path, and the first two the blocked
order with idle workgroups in it, is checked in test_launches.py.  Every
operation of the two paths is the same in the same order, so the tolerance is
zero.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from test_gpu_march import pair  # noqa: E402

CASES = {
    "blocked_fp64": ((120, 122, 6, 66), "fp64"),
    "blocked_fp32": ((120, 190, 6, 66), "fp32"),
    "narrow_fp64": ((40, 60, 40, 8), "fp64"),
    "narrow_fp32": ((40, 60, 40, 8), "fp32"),
}


@pytest.mark.parametrize("dims,storage", list(CASES.values()), ids=list(CASES))
@pytest.mark.parametrize("wall,solid,field", [((0, 0, 0), False, False), ((0, 0, 0), False, True),
                                              ((0, 1, 0), True, False), ((1, 1, 1), True, True)],
                         ids=["periodic", "periodic_field", "spheres", "closed_field"])
def test_steps_of_one_call_equal_single_steps(dims, storage, wall, solid, field):
    A, B = pair(dims, storage, wall, solid, field)
    for n in (6, 7):
        print(f"{storage} {dims} walls {wall} solid {solid} field {field}: {n} steps", flush=True)
        A.step(n)
        for _ in range(n):
            B.step(1)
        assert A.time == B.time
        assert torch.equal(A.populations(), B.populations()), n
    A.close()
    B.close()
