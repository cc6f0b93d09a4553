"""The input transform by 16 tiles where whole tiles lie above, below, left or right of the image, at every alignment of the input."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,K,H,W,r,m,pad,n,one_kernel", [
    (20, 33, 2, 9, 70, 3, 8, 20, 4, True), (16, 40, 2, 30, 11, 3, 6, 13, 3, True), (20, 20, 2, 9, 70, 1, 4, 7, 3, False)])
def test_tiles_outside_the_image(N, C, K, H, W, r, m, pad, n, one_kernel):
    """Layers that run the transform and the GEMM as one kernel: as that, and with the kernel that this test is for."""
    from paper_2007_12216_amd.layer import ConvLayer
    print("wide padding", N, C, K, H, W, r, m, pad, n, flush=True)
    x, w = si.int8_tensor(741, (N, C, H, W)), si.int8_tensor(742, (K, C, r, r))
    ref = direct_conv2d(x, w, pad)
    for flags in (0, rn.FLAG_SEPARATE_KERNELS) if one_kernel else (0,):
        layer = ConvLayer(N, C, K, H, W, r, m, pad, (251, 241, 239, 233)[:n], flags)
        launched = rn.rnswino_plan_describe(layer.plan)
        assert launched["kernels"][0].startswith("k1_input_transform_tiles") and (launched["fused"] is not None) == (one_kernel and not flags)
        layer.set_weights(w)
        for shift in range(4):
            buf = torch.full((x.size + 64,), -77, dtype=torch.int8, device="cuda:0")
            buf[32 + shift:32 + shift + x.size] = torch.from_numpy(x).to("cuda:0").reshape(-1)
            y = layer.forward(buf[32 + shift:32 + shift + x.size].view(N, C, H, W))
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy(), ref)
