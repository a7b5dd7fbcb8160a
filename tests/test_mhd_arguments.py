"""Arguments of the coupled solver's Python entry points, checked before any
device work (no GPU: objects without a lattice behind them)."""
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

from paper_1905_10182_amd.mhd import CoupledMHD  # noqa: E402

SHAPE = (4, 6, 8)  # nz, ny, nx


def test_stencil_current_chosen_after_the_first_step():
    """`current` is a plain attribute: the work array of the stencil current is
    there whenever a step needs it."""
    seen = []
    S = CoupledMHD.__new__(CoupledMHD)
    S.torch, S.dtype, S.shape, S.current = torch, torch.float64, SHAPE, "populations"
    S._u = S._b = S.F = None
    S.velocity = lambda: (None, "u")
    S.fluid = SimpleNamespace(step_velocity=lambda out: out)
    S.mag = SimpleNamespace(device="cpu", step=lambda u: None,
                            lorentz_force=lambda F, u, current, b: seen.append((current, u, b)))
    S.step()
    S.current = "stencil"
    S.step(2)
    S.current = "populations"
    S.step()
    assert [s[:2] for s in seen] == [("populations", "u"), ("stencil", None), ("stencil", None), ("populations", "u")]
    for current, _, b in seen:
        if current == "stencil":
            assert b.shape == (3,) + SHAPE and b.dtype == S.dtype and b.is_contiguous()


def lattice(cls, **attrs):
    lat = cls.__new__(cls)
    lat.torch, lat.dtype, lat.shape, lat.device, lat.handle = torch, torch.float64, SHAPE, torch.device("cpu"), None
    vars(lat).update(attrs)
    return lat


def reached(lat):
    """Stand-ins for the library: a call that passes the checks ends here."""
    def call(*args):
        raise RuntimeError("reached the library")
    names = ("cmlbm_mhd_fields", "cmlbm_step_velocity")
    lat.lib, lat._stream = SimpleNamespace(**{n: call for n in names}), lambda: None
    return lat


def vec(*shape, dtype=torch.float64):
    return torch.zeros(shape or (3,) + SHAPE, dtype=dtype)


@pytest.mark.parametrize("kw", [dict(b=None), dict(b=vec(3, 4, 6, 4)), dict(b=vec(dtype=torch.float32)),
                                dict(b=vec(3, 8, 6, 4).permute(0, 3, 2, 1)), dict(b=vec().to("meta")),
                                dict(b=vec(), F_out=vec(3, 4, 6, 4)), dict(b=vec(), F_out=vec(dtype=torch.float32)),
                                dict(b=vec(), F_out=vec().to("meta")), dict(b="F_out"),
                                dict(current="populations", b=vec(1, 4, 6, 8))],
                         ids=["none", "small", "fp32", "strided", "device", "small_F", "fp32_F", "device_F", "same",
                              "populations"])
def test_lorentz_force_refuses_work_arrays_that_the_kernels_would_overrun(kw):
    from paper_1905_10182_amd.mhd import MagneticLattice
    mag = reached(lattice(MagneticLattice))
    kw = dict(dict(F_out=vec(), current="stencil"), **kw)
    if isinstance(kw["b"], str):
        kw["b"] = kw["F_out"]
    with pytest.raises(ValueError):
        mag.lorentz_force(**kw)


def test_lorentz_force_takes_what_the_library_takes():
    from paper_1905_10182_amd.mhd import MagneticLattice
    mag = reached(lattice(MagneticLattice))
    for kw in (dict(current="stencil", b=vec()), dict(current="stencil", b=vec(3, 1, *SHAPE)), dict(),
               dict(u=vec()), dict(u=vec(), b=vec())):
        with pytest.raises(RuntimeError, match="reached the library"):
            mag.lorentz_force(vec(3, 1, *SHAPE), **kw)


@pytest.mark.parametrize("out", [vec().to("meta"), vec(3, 4, 6, 8)[..., :7], vec(3, 2, 6, 8), vec(dtype=torch.float16)],
                         ids=["device", "strided", "small", "fp16"])
def test_step_velocity_refuses_what_the_kernel_would_overrun(out):
    from paper_1905_10182_amd import Lattice
    fluid = reached(lattice(Lattice))
    with pytest.raises((ValueError, AssertionError)):
        fluid.step_velocity(out)


def test_step_velocity_takes_both_types():
    from paper_1905_10182_amd import Lattice
    fluid = reached(lattice(Lattice))
    for dtype in (torch.float64, torch.float32):
        with pytest.raises(RuntimeError, match="reached the library"):
            fluid.step_velocity(vec(dtype=dtype))
