"""ConvLayer and ConvStack on a stream that is current but not the default one: their kernels have to queue behind the work that is already on
it.  The inputs arrive late there: work of some milliseconds goes first, and on any other stream the kernels would read zeros."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import direct_conv2d
from paper_2007_12216_amd.layer import ConvLayer
from paper_2007_12216_amd.stack import ConvStack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def busy():
    return torch.zeros(1 << 27, dtype=torch.float32, device="cuda:0")


def behind_other_work(call, source, busy):
    """call(x) on a side stream, x a device tensor that holds zeros until the stream has worked off 60 passes over `busy`.  Taken again, at
    most twice, if the host was held up for so long that the stream was idle when the call returned."""
    side = torch.cuda.Stream()                               # default priority
    for _ in range(3):
        x = torch.zeros_like(source)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(60):
                busy.add_(1.0)
            x.copy_(source)
            out = call(x)
            at_work = not side.query()
        side.synchronize()
        if at_work:
            return out
    pytest.fail("the stream never had work left when the call returned")


@pytest.mark.parametrize("device", ["cuda:0", "cuda"])       # the stream is found with and without a device index
def test_layer_follows_the_current_stream(device, busy):
    print("layer on a side stream", device, flush=True)
    N, C, K, H, W, r, m, pad, moduli = 2, 70, 40, 28, 28, 3, 8, 1, (251, 241, 239, 233)
    x, w = si.int8_tensor(91, (N, C, H, W)), si.int8_tensor(92, (K, C, r, r))
    xd, wd = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    layer = ConvLayer(N, C, K, H, W, r, m, pad, moduli, device=device)
    ref = direct_conv2d(x, w, pad)

    def late_weights(weights):
        layer.set_weights(weights)
        return layer.forward(xd)

    assert np.array_equal(behind_other_work(late_weights, wd, busy).cpu().numpy(), ref)
    layer.y.zero_()
    assert np.array_equal(behind_other_work(layer.forward, xd, busy).cpu().numpy(), ref)


def test_stack_follows_the_current_stream(busy):
    print("stack on a side stream", flush=True)
    layers = si.vgg16_stack(batch=1, hw=32)
    stack = ConvStack(layers)
    stack.set_weights([si.int8_tensor(l["seed_w"], (l["K"], l["C"], l["r"], l["r"])) for l in layers])
    xd = torch.from_numpy(si.int8_tensor(si.VGG16_SEED_X, (1, 3, 32, 32))).to("cuda:0")
    stack.forward(xd)
    want = [a.cpu().numpy().copy() for a in stack.act]
    assert all((a != 0).mean() > 0.5 for a in want)
    for a in stack.act:
        a.zero_()
    assert behind_other_work(stack.forward, xd, busy) is stack.act[-1]
    assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(stack.act, want))
