"""The row-tiled convolution against the brick-tiled one and the FP64 oracle.

A batch large enough takes the row kernel; the same samples in batches of too
few workgroups take the brick kernel.  Both add an output's products in the
same order, so the outputs are the same bits.  Two samples are also held
against the oracle, within one BF16 ulp plus 1e-5 of the accumulated magnitude
(the bound of the brick kernel's own test).
"""
import numpy as np
import pytest

from oracle import conv_oracle as C
import workloads as W

pytestmark = pytest.mark.gpu

# (n, d, h, w), cin, cout, periodic; row workgroups = n * d/4 * h/8 * w/16 * cout/32
CASES = [((192, 4, 8, 16), 32, 32, (1, 1, 1)),   # the rule's edge; a brick that wraps onto itself
         ((25, 4, 16, 16), 96, 128, (0, 1, 0)),  # three input chunks, four output blocks, padding
         ((17, 8, 8, 32), 160, 96, (1, 0, 0)),   # 204 workgroups: no multiple of the 8 XCDs
         ((3, 16, 24, 96), 32, 32, (0, 0, 1))]   # 216 bricks, interior and edge ones


@pytest.mark.parametrize("dims,cin,cout,per", CASES)
@pytest.mark.parametrize("act", [0, 1])
def test_rows_match_bricks(dims, cin, cout, per, act):
    import torch
    from paper_1905_10182_amd import cmnn as nn
    print("conv rows", dims, cin, cout, per, act, flush=True)
    n, d, h, w = dims
    rng = W.generator(11)

    def bf16(shape, scale=1.0):
        return torch.as_tensor((rng.standard_normal(shape) * scale).astype(np.float32)).to(torch.bfloat16).cuda()

    x, gate = bf16(dims + (cin,)), bf16(dims + (cout,))
    wt = bf16((27, cout, cin), 0.1)
    bias = torch.as_tensor(rng.standard_normal(cout) * 0.1, dtype=torch.float32, device="cuda:0")

    def run(lo, hi, forward, pad=0):
        buf = torch.full(((hi - lo) * d * h * w * cout + pad,), 7.0, dtype=torch.bfloat16, device="cuda:0")
        y = buf[pad:].view((hi - lo, d, h, w, cout))
        g = nn.geom(hi - lo, d, h, w, periodic=per)
        if forward:
            nn.conv_fwd(g, x[lo:hi], cin, wt, bias, cout, act, y)
        elif act:
            nn.conv_bwd_data_act(g, x[lo:hi], cin, wt, cout, gate[lo:hi], act, y)
        else:
            nn.conv_bwd_data(g, x[lo:hi], cin, wt, cout, y)
        return y

    blocks = d // 4 * (h // 8) * (w // 16) * (cout // 32)
    few = max(1, 191 // blocks)
    f64 = [t.float().cpu().numpy().astype(np.float64) for t in (x[[0, n - 1]], wt)]
    for forward in (True, False):
        y = run(0, n, forward)
        for lo in range(0, n, few):
            hi = min(n, lo + few)
            assert torch.equal(y[lo:hi], run(lo, hi, forward)), (forward, lo)
        # an output that is not 8-byte aligned takes the brick kernel
        assert torch.equal(y, run(0, n, forward, pad=1))
        if forward:
            ref = C.conv3d(f64[0], f64[1], bias.cpu().numpy().astype(np.float64), per)
            if act:
                ref = C.leaky(ref)
            mag = C.conv3d(np.abs(f64[0]), np.abs(f64[1]), None, per)
            err = np.abs(y[[0, n - 1]].float().cpu().numpy() - ref)
            assert (err <= np.abs(ref) * 2.0 ** -8 + 1e-5 * mag + 1e-30).all()
