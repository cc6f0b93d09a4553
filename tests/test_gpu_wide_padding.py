"""The 16-tile input transform where whole tiles lie above, below, left or right of the image, at every alignment of the input."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,K,H,W,r,m,pad,n", [(20, 33, 2, 9, 70, 3, 8, 20, 4), (16, 40, 2, 30, 11, 3, 6, 13, 3), (20, 20, 2, 9, 70, 1, 4, 7, 3)])
def test_tiles_outside_the_image(N, C, K, H, W, r, m, pad, n):
    from paper_2007_12216_amd.layer import ConvLayer
    print("wide padding", N, C, K, H, W, r, m, pad, n, flush=True)
    x, w = si.int8_tensor(741, (N, C, H, W)), si.int8_tensor(742, (K, C, r, r))
    layer = ConvLayer(N, C, K, H, W, r, m, pad, (251, 241, 239, 233)[:n])
    assert rn.rnswino_plan_describe(layer.plan)["kernels"][0].startswith("k1_input_transform_tiles")
    layer.set_weights(w)
    ref = direct_conv2d(x, w, pad)
    for shift in range(4):
        buf = torch.full((x.size + 64,), -77, dtype=torch.int8, device="cuda:0")
        buf[32 + shift:32 + shift + x.size] = torch.from_numpy(x).to("cuda:0").reshape(-1)
        y = layer.forward(buf[32 + shift:32 + shift + x.size].view(N, C, H, W))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), ref)
