"""Eight steps in one pass of k2_march with two FP32 cells a lane, and rows of
exactly one such strip: cmlbm2d_step(n) gives the same bits as n calls of one
step, which run k2_step alone.  That these planes take those passes is checked in
test_launches.py.  Every operation is the same in the same order, so the
tolerance is zero.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

import test_gpu_march2d_long  # noqa: E402

DIMS = [(8192, 1750), (5000, 3750), (128, 70000)]


@pytest.mark.parametrize("force", ["uniform", "field"])
@pytest.mark.parametrize("dims", DIMS, ids=[f"{a}x{b}" for a, b in DIMS])
def test_eight_fp32_steps_equal_single_steps(dims, force):
    test_gpu_march2d_long.test_long_passes_equal_single_steps(dims, "fp32", force)
