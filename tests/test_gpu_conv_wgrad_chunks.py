"""The brick-tiled weight gradient over chunks of several bricks, against the
FP64 oracle.

Shapes where a workgroup loops: chunks of four bricks with a shorter last one
that cross rows, planes and samples of bricks, more than one output and input
tile, every padding.  BF16 products are exact in FP32, so only the order of the
FP32 sums differs from the oracle: within 1e-5 relative, as for a single brick.
"""
import numpy as np
import pytest

from oracle import conv_oracle as C
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,cin,cout,per", [((3, 12, 20, 48), 96, 64, (0, 1, 0)), ((2, 20, 16, 80), 64, 96, (1, 0, 1)),
                                               ((5, 4, 24, 32), 64, 256, (0, 0, 0))])
def test_chunks_of_bricks(dims, cin, cout, per):
    import torch
    from paper_1905_10182_amd import cmnn as nn
    print("conv wgrad", dims, cin, cout, per, flush=True)
    rng = W.generator(12)

    def bf16(shape):
        t = torch.as_tensor(rng.standard_normal(shape).astype(np.float32)).to(torch.bfloat16).cuda()
        return t, t.float().cpu().numpy().astype(np.float64)

    g = nn.geom(*dims, periodic=per)
    x, xr = bf16(dims + (cin,))
    dy, dyr = bf16(dims + (cout,))
    ws = torch.empty(nn.conv_bwd_weight_workspace(g, cin, cout) // 4, dtype=torch.float32, device="cuda:0")
    dw = torch.empty((27, cout, cin), dtype=torch.float32, device="cuda:0")
    db = torch.empty((cout,), dtype=torch.float32, device="cuda:0")
    nn.conv_bwd_weight(g, x, cin, dy, cout, dw, db, ws)
    _, rdw, rdb = C.conv3d_grads(xr, np.zeros((27, cout, cin)), dyr, per)
    assert np.linalg.norm(dw.cpu().numpy() - rdw) < 1e-5 * np.linalg.norm(rdw)
    assert np.linalg.norm(db.cpu().numpy() - rdb) < 1e-5 * np.linalg.norm(rdb)
    dw2 = torch.empty_like(dw)
    nn.conv_bwd_weight(g, x, cin, dy, cout, dw2, None, ws)
    assert torch.equal(dw, dw2)  # deterministic, and without a bias gradient
