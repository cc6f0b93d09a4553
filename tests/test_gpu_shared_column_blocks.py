"""The input transform of a few blocks, where two blocks share a residue's column blocks: tiles of 12 to 16 points a side (9 to 16 column
blocks, so that the second block has one to eight), both widths, several residues, packed tiles, up to the line (128 blocks) and past it; and
layers of a single residue, whose blocks never share."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu

THREE, WIDE = (251, 241, 239), (65521, 65519)


@pytest.mark.parametrize("N,C,K,H,W,r,m,moduli,sharing", [
    (1, 5, 3, 20, 20, 3, 10, THREE, 2), (1, 5, 3, 23, 20, 3, 11, THREE[:1], 1), (1, 30, 3, 25, 13, 3, 12, WIDE, 2), (1, 70, 5, 27, 40, 3, 13, THREE, 2),
    (1, 40, 3, 28, 28, 3, 14, THREE, 2), (1, 66, 3, 40, 41, 3, 14, WIDE, 2), (2, 33, 3, 45, 60, 3, 10, WIDE[:1], 1),
    (2, 128, 3, 56, 56, 3, 14, WIDE[:1] + (65497,), 2), (2, 128, 3, 56, 57, 3, 14, WIDE, 1),
    (2, 20, 3, 40, 40, 3, 10, THREE, 2), (2, 20, 3, 40, 40, 3, 10, WIDE, 2), (2, 20, 3, 56, 56, 3, 14, THREE, 2), (2, 10, 3, 56, 56, 3, 13, WIDE, 2)])
def test_two_blocks_share_the_column_blocks(N, C, K, H, W, r, m, moduli, sharing):
    from paper_2007_12216_amd.layer import ConvLayer
    print("shared column blocks", N, C, K, H, W, r, m, moduli, flush=True)
    x, w = si.int8_tensor(751, (N, C, H, W)), si.int8_tensor(752, (K, C, r, r))
    layer = ConvLayer(N, C, K, H, W, r, m, 1, moduli, rn.FLAG_ALLOW_UNCHECKED_RANGE)
    extents = rn.rnswino_plan_describe(layer.plan)["grids"][0].split("x")
    assert (int(extents[2]) if len(extents) > 2 else 1) == sharing
    layer.set_weights(w)
    layer.workspace.fill_(0x55)                        # a column block that nobody writes shows
    y = layer.forward(torch.from_numpy(x).to("cuda:0"))
    torch.cuda.synchronize()
    P = int(np.prod([int(p) for p in moduli]))
    ref = direct_conv2d(x, w, 1).astype(np.int64)
    ref = (ref + (P - 1) // 2) % P - (P - 1) // 2      # the symmetric range of the moduli, where it is the smaller
    assert np.array_equal(y.cpu().numpy().astype(np.int64), ref)
