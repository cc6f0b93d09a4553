"""The input transform's 16-byte row segments at the ends of the tensor: tensors smaller than a segment, rows shorter than one,
wide padding, packed tiles, and an input at every alignment between other data that must not leak in."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu

THREE, WIDE = (251, 241, 239), (65521, 65519)


@pytest.mark.parametrize("N,C,K,H,W,r,m,pad,moduli", [
    (1, 1, 1, 1, 1, 1, 2, 0, THREE), (1, 1, 2, 3, 3, 3, 4, 1, THREE), (1, 1, 1, 3, 5, 3, 8, 1, THREE), (1, 2, 3, 2, 4, 3, 8, 2, THREE),
    (1, 1, 2, 4, 4, 5, 12, 2, WIDE), (1, 1, 1, 2, 9, 3, 8, 5, THREE), (2, 5, 3, 4, 5, 3, 8, 1, THREE), (1, 3, 2, 1, 40, 3, 10, 1, THREE),
    (1, 65, 3, 3, 16, 3, 14, 1, WIDE), (1, 2, 2, 15, 1, 3, 8, 1, THREE), (1, 40, 2, 9, 17, 3, 8, 20, THREE), (2, 3, 4, 33, 33, 3, 8, 1, THREE),
    (16, 1, 2, 7, 9, 3, 4, 3, THREE), (1, 16, 3, 47, 35, 5, 12, 2, THREE)])
def test_segments_at_the_ends_of_the_tensor(N, C, K, H, W, r, m, pad, moduli):
    from paper_2007_12216_amd.layer import ConvLayer
    print("input edges", N, C, K, H, W, r, m, pad, moduli, flush=True)
    x, w = si.int8_tensor(721, (N, C, H, W)), si.int8_tensor(722, (K, C, r, r))
    layer = ConvLayer(N, C, K, H, W, r, m, pad, moduli)
    layer.set_weights(w)
    ref = direct_conv2d(x, w, pad)
    for shift in (0, 1, 7, 15):
        buf = torch.full((x.size + 64,), -77, dtype=torch.int8, device="cuda:0")
        buf[32 + shift:32 + shift + x.size] = torch.from_numpy(x).to("cuda:0").reshape(-1)
        y = layer.forward(buf[32 + shift:32 + shift + x.size].view(N, C, H, W))
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), ref)


@pytest.mark.parametrize("N,C,K,H,W,r,m,pad,moduli,one_kernel", [
    (5, 65, 2, 50, 51, 3, 8, 1, THREE[:2] + (239, 233), False),         # two channel blocks, the second with one channel
    (4, 70, 3, 57, 43, 3, 6, 1, THREE + (233,), False),                 # 8 contraction slots a row, t * t a multiple of 16
    (9, 64, 2, 50, 47, 3, 7, 0, THREE + (233,), True),                 # t = 9: a last block of one point, ragged tiles and tile block
    (11, 40, 2, 31, 23, 1, 4, 0, THREE, False),                         # 1 x 1 filter, one full block of points
    (9, 64, 2, 21, 22, 1, 3, 0, THREE, False),                          # t = 3: no full block of points
    (171, 33, 2, 17, 18, 3, 8, 3, THREE, True),                        # several images in one block of tiles, wide padding
    (1, 64, 2, 150, 161, 3, 8, 1, THREE + (233,), True),               # a residue per block
    (10, 3, 4, 200, 211, 3, 8, 1, THREE + (233,), False), (9, 17, 3, 75, 77, 3, 6, 1, THREE, False)])     # packed tiles, ragged last slot
def test_sixteen_tiles_at_a_time(N, C, K, H, W, r, m, pad, moduli, one_kernel):
    """Layers that run the transform and the GEMM as one kernel: as that, and with the kernel that this test is for."""
    from paper_2007_12216_amd.layer import ConvLayer
    print("sixteen tiles", N, C, K, H, W, r, m, pad, moduli, flush=True)
    x, w = si.int8_tensor(731, (N, C, H, W)), si.int8_tensor(732, (K, C, r, r))
    ref = direct_conv2d(x, w, pad)
    for flags in (0, rn.FLAG_SEPARATE_KERNELS) if one_kernel else (0,):
        layer = ConvLayer(N, C, K, H, W, r, m, pad, moduli, flags)
        launched = rn.rnswino_plan_describe(layer.plan)
        assert launched["kernels"][0].startswith("k1_input_transform_tiles") and (launched["fused"] is not None) == (one_kernel and not flags)
        layer.set_weights(w)
        for shift in (0, 5):
            buf = torch.full((x.size + 64,), -77, dtype=torch.int8, device="cuda:0")
            buf[32 + shift:32 + shift + x.size] = torch.from_numpy(x).to("cuda:0").reshape(-1)
            y = layer.forward(buf[32 + shift:32 + shift + x.size].view(N, C, H, W))
            torch.cuda.synchronize()
            assert np.array_equal(y.cpu().numpy(), ref)
