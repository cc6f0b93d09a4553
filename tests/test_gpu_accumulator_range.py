"""The input transform's accumulators at the largest magnitude its table can reach: an accumulator that starts at
0x4B400000 + a is read as a binary32 number, which holds as long as |a + sum| stays below 2^22."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu


# one image per modulus (blocks of one tile), and many images (blocks of 16 tiles: all residues in one, one residue each with packed channels)
@pytest.mark.parametrize("images,C", [(0, 16), (800, 64), (1600, 16)])
@pytest.mark.parametrize("m,moduli", [(8, (251, 241, 239)), (8, (253, 251, 247)), (14, (251, 241, 239)), (2, (3, 5, 7, 11, 13, 17, 19, 23))])
@pytest.mark.parametrize("sign", [1, -1])
def test_tiles_that_drive_one_transform_point_to_its_largest_sum(m, moduli, sign, images, C):
    from paper_2007_12216_amd.layer import ConvLayer
    r, t, K, N = 3, m + 2, 16, images or len(moduli)
    print("accumulator range", m, moduli, sign, N, C, flush=True)
    layer = ConvLayer(N, C, K, t, t, r, m, 0, moduli, flags=rn.FLAG_ALLOW_UNCHECKED_RANGE)
    sixteen = rn.rnswino_plan_describe(layer.plan)["kernels"][0].startswith("k1_input_transform_tiles")
    assert sixteen == (images > 0 and t <= 10)
    x = np.empty((N, C, t, t), dtype=np.int8)
    for i in range(len(moduli)):
        bt = rn.rnswino_plan_get_matrix(layer.plan, rn.MATRIX_BT, i).astype(np.int64)
        kron = np.einsum("ab,cd->acbd", bt, bt).reshape(t * t, t * t)
        p = moduli[i]
        kron = (kron + (p - 1) // 2) % p - (p - 1) // 2
        row = kron[np.abs(kron).sum(axis=1).argmax()].reshape(t, t)          # the worst row of modulus i, in every len(moduli)-th image
        x[i::len(moduli)] = np.where(sign * row > 0, 127, -128)
    w = si.int8_tensor(611, (K, C, r, r))
    w = (w // 32).astype(np.int8) if np.prod([float(p) for p in moduli]) < 1e8 else w     # inside the range of the set
    layer.set_weights(w)
    y = layer.forward(torch.from_numpy(x).to("cuda:0"))
    torch.cuda.synchronize()
    ref = direct_conv2d(x, w, 0).astype(np.int64)
    P = int(np.prod([int(p) for p in moduli], dtype=object))
    half = (P - 1) // 2
    want = ref if P > 1 << 33 else (ref + half) % P - half
    assert np.array_equal(y.cpu().numpy().astype(np.int64), want)
