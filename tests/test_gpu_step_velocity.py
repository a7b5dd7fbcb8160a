"""cmlbm_step_velocity against the moment export followed by a step: the same
velocity and the same populations, bit for bit, on the fused route (a force
field, the method's collision, io type = storage) and on every other one."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from paper_1905_10182_amd import Lattice  # noqa: E402

CASES = [dict(), dict(wall=(0, 1, 0), solid=True), dict(model="m4"), dict(rho0=1.1), dict(field=False), dict(other_io=True)]


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp16"])
@pytest.mark.parametrize("case", CASES, ids=["fused", "walls", "m4", "rho0", "uniform", "other_io"])
def test_velocity_and_step_match_export_then_step(storage, case):
    case = dict(case)
    field, other_io = case.pop("field", True), case.pop("other_io", False)
    if storage == "fp16" and "model" in case:
        pytest.skip("comparison models are for FP64 and FP32 storage")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    lats = []
    for _ in range(2):
        lat = Lattice(70, 13, 9, nbatch=2, tau=0.7, storage=storage, device="cuda:0", **case)
        lats.append(lat)
    shape = lats[0].shape
    f = (0.8 + 0.4 * torch.rand((27,) + shape, generator=g, device="cuda", dtype=torch.float64)) / 27
    F = 1e-3 * (torch.rand((3,) + shape, generator=g, device="cuda", dtype=torch.float64) - 0.5)
    S = torch.rand(shape, generator=g, device="cuda") < 0.1
    for lat in lats:
        if case.get("solid"):
            lat.set_solid(S)
        if field:
            lat.set_force("field", field=F)
        else:
            lat.set_force("uniform", [1e-4, 2e-5, -3e-5])
        lat.load_populations(f)
    A, B = lats
    dt = torch.float64 if (storage == "fp64") != other_io else torch.float32
    for _ in range(3):
        u = A.step_velocity(torch.full((3,) + shape, 9.0, dtype=dt, device="cuda"))
        ref = B.moments(dtype=dt)[1]
        B.step(1)
        assert torch.equal(u, ref)
        assert A.time == B.time and torch.equal(A.populations(), B.populations())
