"""The input transform's accumulators at the largest magnitude its table can reach: an accumulator that starts at
0x4B400000 + a is read as a binary32 number, which holds as long as |a + sum| stays below 2^22."""
import numpy as np
import pytest
import torch

import synth_inputs as si
import paper_2007_12216_amd as rn
from oracle import direct_conv2d

pytestmark = pytest.mark.gpu


# one tile per modulus (blocks of one tile), and many images of 2 x 2 tiles (blocks of 16 tiles, also with packed channels: all residues
# in one for the tiles of 8, one residue each for those of 2), each with one tile that drives the sum, in every lane of a block in turn
@pytest.mark.parametrize("images,C", [(0, 16), (384, 64), (1536, 16)])
@pytest.mark.parametrize("m,moduli", [(8, (251, 241, 239)), (8, (253, 251, 247)), (14, (251, 241, 239)), (2, (3, 5, 7, 11, 13, 17, 19, 23))])
@pytest.mark.parametrize("sign", [1, -1])
def test_tiles_that_drive_one_transform_point_to_its_largest_sum(m, moduli, sign, images, C):
    """Layers of 64 channels run the transform and the GEMM as one kernel (t <= 10): as that, and with the input transform of its own."""
    N = (images if m == 8 else images // 4) if images else len(moduli)
    one_kernel = C == 64 and m <= 8
    for flags in (0, rn.FLAG_SEPARATE_KERNELS) if one_kernel else (0,):
        launched = _drive(m, moduli, sign, N, C, 16, 2 if images else 1, flags)
        assert launched["kernels"][0].startswith("k1_input_transform_tiles") == (images > 0 and m <= 8)
        assert (launched["fused"] is not None) == (one_kernel and not flags)


# the other forms of that kernel: three and four contraction steps, and packed channels
@pytest.mark.parametrize("m,N,C,K,kernel", [(10, 240, 64, 16, "k12_transform_gemm<3, 1, 1, false>"), (14, 320, 64, 16, "k12_transform_gemm<4, 1, 1, false>"),
                                            (8, 1024, 4, 64, "k12_transform_gemm<2, 2, 1, true>")])
@pytest.mark.parametrize("sign", [1, -1])
def test_the_largest_sum_in_one_kernel_with_the_gemm(m, N, C, K, kernel, sign):
    assert _drive(m, (251, 241, 239), sign, N, C, K, 2, 0)["fused"] == kernel


def _drive(m, moduli, sign, N, C, K, side, flags):
    """N images of side x side tiles through a layer, against the oracle; returns the report of what was launched."""
    from paper_2007_12216_amd.layer import ConvLayer
    r, t = 3, m + 2
    H = t + (side - 1) * m
    print("accumulator range", m, moduli, sign, N, C, flags, flush=True)
    layer = ConvLayer(N, C, K, H, H, r, m, 0, moduli, flags=flags | rn.FLAG_ALLOW_UNCHECKED_RANGE)
    x = si.int8_tensor(612, (N, C, H, H))
    for i in range(len(moduli)):
        bt = rn.rnswino_plan_get_matrix(layer.plan, rn.MATRIX_BT, i).astype(np.int64)
        kron = np.einsum("ab,cd->acbd", bt, bt).reshape(t * t, t * t)
        p = moduli[i]
        kron = (kron + (p - 1) // 2) % p - (p - 1) // 2
        row = kron[np.abs(kron).sum(axis=1).argmax()].reshape(t, t)          # the worst row of modulus i, in every len(moduli)-th image
        for img in range(i, N, len(moduli)):
            j, k = divmod(img // len(moduli) % 4, 2) if side > 1 else (0, 0)
            x[img, :, j * m:j * m + t, k * m:k * m + t] = np.where(sign * row > 0, 127, -128)
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
    return rn.rnswino_plan_describe(layer.plan)
