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
