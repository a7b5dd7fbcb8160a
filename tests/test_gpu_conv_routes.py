"""The brick-tiled convolution in its wide output tiles, and the two ends of the
small-grid kernel's range, against the same samples in small batches and the
FP64 oracle.

All kernels add an output's products in the same order, so a large batch gives
the same bits as its samples in batches that take another kernel (which kernel
a size takes is checked in test_launches.py).  Two samples are also held
against the oracle, within one BF16 ulp plus 1e-5 of the accumulated magnitude.
"""
import numpy as np
import pytest

from oracle import conv_oracle as C
import workloads as W

pytestmark = pytest.mark.gpu

# (n, d, h, w), input and output channels, periodic, samples of a small batch
CASES = {
    "tile4": ((32, 16, 4, 64), 32, 64, (1, 0, 1), 1),    # 512 workgroups of 64 channels; batches: 16-channel tiles
    "tile6": ((33, 16, 4, 64), 96, 96, (0, 1, 0), 2),    # 528 workgroups of 96, three input chunks; batches: k_conv_few
    "few_1": ((2, 4, 4, 16), 64, 32, (1, 1, 1), 1),      # one brick that wraps onto itself
    "few_edge": ((16, 8, 12, 16), 32, 64, (0, 0, 0), 4),  # one input chunk, 192 workgroups; batches: 16-channel tiles
}


@pytest.mark.parametrize("dims,cin,cout,per,few", list(CASES.values()), ids=list(CASES))
@pytest.mark.parametrize("act", [0, 1])
def test_large_batches_match_small_ones(dims, cin, cout, per, few, act):
    import torch
    from paper_1905_10182_amd import cmnn as nn
    print("conv routes", dims, cin, cout, per, act, flush=True)
    n = dims[0]
    rng = W.generator(17)

    def bf16(shape, scale=1.0):
        return torch.as_tensor((rng.standard_normal(shape) * scale).astype(np.float32)).to(torch.bfloat16).cuda()

    x, gate, wt = bf16(dims + (cin,)), bf16(dims + (cout,)), bf16((27, cout, cin), 0.1)
    bias = torch.as_tensor(rng.standard_normal(cout) * 0.1, dtype=torch.float32, device="cuda:0")

    def run(lo, hi, forward, pad=0):
        shape = (hi - lo,) + dims[1:]
        buf = torch.full((int(np.prod(shape)) * cout + pad,), 7.0, dtype=torch.bfloat16, device="cuda:0")
        y = buf[pad:].view(shape + (cout,))
        g = nn.geom(*shape, periodic=per)
        if forward:
            nn.conv_fwd(g, x[lo:hi], cin, wt, bias, cout, act, y)
        elif act:
            nn.conv_bwd_data_act(g, x[lo:hi], cin, wt, cout, gate[lo:hi], act, y)
        else:
            nn.conv_bwd_data(g, x[lo:hi], cin, wt, cout, y)
        return y

    pick = [0, n - 1]
    xr, wr = (t.float().cpu().numpy().astype(np.float64) for t in (x[pick], wt))
    for forward in (True, False):
        y = run(0, n, forward)
        assert torch.equal(y, run(0, n, forward, pad=1))  # not 8-byte aligned: bricks
        for lo in range(0, n, few):
            assert torch.equal(y[lo:lo + few], run(lo, min(n, lo + few), forward)), (forward, lo)
        if forward:
            ref = C.conv3d(xr, wr, bias.cpu().numpy().astype(np.float64), per)
            if act:
                ref = C.leaky(ref)
            mag = C.conv3d(np.abs(xr), np.abs(wr), None, per)
            err = np.abs(y[pick].float().cpu().numpy() - ref)
            assert (err <= np.abs(ref) * 2.0 ** -8 + 1e-5 * mag + 1e-30).all()
