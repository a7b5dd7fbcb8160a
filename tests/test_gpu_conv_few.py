"""The convolution of small grids (k_conv_few) against the brick-tiled one and
the FP64 oracle.

An output that is not 8-byte aligned takes the brick kernel, an aligned one the
kernel under test; both add an output's products in the same order, so the
outputs are the same bits.  One sample is also held against the oracle, within
one BF16 ulp plus 1e-5 of the accumulated magnitude (the brick kernel's bound).
Input channels in one, two, three and six chunks; a single brick that wraps onto
itself, every padding, several samples, more workgroups than CUs.
"""
import numpy as np
import pytest

from oracle import conv_oracle as C
import workloads as W

pytestmark = pytest.mark.gpu

CASES = [((1, 4, 4, 16), 32, 32, (1, 1, 1)), ((2, 8, 4, 32), 64, 96, (0, 1, 0)), ((3, 4, 12, 16), 96, 32, (1, 0, 1)),
         ((2, 8, 8, 16), 192, 64, (0, 0, 0)), ((7, 4, 20, 64), 64, 64, (1, 0, 0))]


@pytest.mark.parametrize("dims,cin,cout,per", CASES)
@pytest.mark.parametrize("act", [0, 1])
def test_small_grids_match_bricks(dims, cin, cout, per, act):
    import torch
    from paper_1905_10182_amd import cmnn as nn
    print("conv few", dims, cin, cout, per, act, flush=True)
    rng = W.generator(13)

    def bf16(shape, scale=1.0):
        return torch.as_tensor((rng.standard_normal(shape) * scale).astype(np.float32)).to(torch.bfloat16).cuda()

    x, gate, wt = bf16(dims + (cin,)), bf16(dims + (cout,)), bf16((27, cout, cin), 0.1)
    bias = torch.as_tensor(rng.standard_normal(cout) * 0.1, dtype=torch.float32, device="cuda:0")
    g = nn.geom(*dims, periodic=per)

    def run(forward, pad, b):
        buf = torch.full((int(np.prod(dims)) * cout + pad,), 7.0, dtype=torch.bfloat16, device="cuda:0")
        y = buf[pad:].view(dims + (cout,))
        if forward:
            nn.conv_fwd(g, x, cin, wt, b, cout, act, y)
        elif act:
            nn.conv_bwd_data_act(g, x, cin, wt, cout, gate, act, y)
        else:
            nn.conv_bwd_data(g, x, cin, wt, cout, y)
        return y

    y = run(True, 0, bias)
    assert torch.equal(y, run(True, 1, bias))
    assert torch.equal(run(True, 0, None), run(True, 1, None))
    assert torch.equal(run(False, 0, None), run(False, 1, None))
    xr, wr = (t.float().cpu().numpy().astype(np.float64) for t in (x[-1:], wt))
    ref = C.conv3d(xr, wr, bias.cpu().numpy().astype(np.float64), per)
    if act:
        ref = C.leaky(ref)
    mag = C.conv3d(np.abs(xr), np.abs(wr), None, per)
    err = np.abs(y[-1:].float().cpu().numpy() - ref)
    assert (err <= np.abs(ref) * 2.0 ** -8 + 1e-5 * mag + 1e-30).all()
