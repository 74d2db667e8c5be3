"""Every block tile of the warm-start network's 3x3 convolutions.  The tile
follows from the number of positions (samples x (S + 1)^2), so batches as large
as those in use take tiles that a few samples never reach: four or eight waves,
32 or 64 channels, 128 to 512 positions a block.

Forward: small integers and weights of +-1, exact in any order, so the outputs
equal plain torch in float64 (with the same roundings of activations to
bfloat16) to the last bit.  Gradients: a batch split in halves, quarters, ... of
samples down to two runs through the small tiles; with a power of two of parts
the output gradients differ by an exact factor, every rounding to bfloat16 falls
alike, and the sums of the parts' gradients agree to float32 summation."""
import numpy as np
import pytest
import torch
import torch.nn.functional as nnf

from test_gpu_dmnet_chunks import DEV, exact_case
from oracle import cnn_oracle as net

pytestmark = pytest.mark.gpu


def torch_forward(params, x):
    """the two-level network in float64, inputs of the 3x3 convolutions rounded
    to bfloat16"""
    w = [torch.from_numpy(np.ascontiguousarray(p)) for p in params]

    def conv(i, h):
        h = h.to(torch.bfloat16).double()
        return torch.relu(nnf.conv2d(h, w[2 * i], w[2 * i + 1], padding=1))

    skip = conv(1, conv(0, torch.from_numpy(x)))
    h = conv(3, conv(2, nnf.avg_pool2d(skip, 2)))
    u = torch.cat([nnf.interpolate(h, scale_factor=2, mode="nearest"), skip], 1)
    return nnf.conv2d(conv(5, conv(4, u)), w[12], w[13])


def network(n, size, c0, params):
    from paper_1808_10375_amd import dmnet
    m = dmnet.DMNet(n, size=size, base_ch=c0, levels=2, device=DEV)
    m.set_params(net.flatten(params))
    return m


# (tiles as <channels of a wave / 16, positions of a wave / 16, waves side by side
# in channels, waves>) <2,4,1,4> and <2,4,1,8>; those and <2,4,2,4>; <4,4,1,4>,
# <2,4,2,4> and <2,4,2,8>; the same with sample counts and rows that fill no
# block of positions
@pytest.mark.parametrize("n,size,c0", [(32, 64, 32), (64, 64, 32), (128, 32, 64), (35, 62, 32),
                                       (67, 62, 32), (131, 32, 64), (45, 54, 64)])
def test_forward_of_large_batches_exact(n, size, c0):
    print(f"case conv tiles forward n={n} size={size} base={c0}", flush=True)
    params, x, _ = exact_case(n + size + c0, n, size, c0, 2)
    y = network(n, size, c0, params).forward(torch.from_numpy(x).float().to(DEV)).cpu()
    want = torch_forward(params, x)
    assert want.abs().max() < 2 ** 21
    assert torch.equal(y, want.float())


@pytest.mark.parametrize("n,size,c0", [(32, 64, 32), (64, 32, 64), (128, 32, 64)])
def test_gradients_of_large_batches_equal_their_parts(n, size, c0):
    print(f"case conv tiles gradients n={n} size={size} base={c0}", flush=True)
    params, x, target = exact_case(n + size + c0, n, size, c0, 2)
    x, target = (torch.from_numpy(a).float().to(DEV) for a in (x, target))
    loss, g = network(n, size, c0, params).loss_grad(x, target)
    small = network(2, size, c0, params)
    parts = [small.loss_grad(x[i:i + 2], target[i:i + 2]) for i in range(0, n, 2)]
    want = sum(p[1].double() for p in parts) / (n // 2)
    assert abs(loss - np.mean([p[0] for p in parts])) <= 1e-5 * abs(loss)
    # float32 sums of up to n size^2 products against the float64 sum of parts
    assert float((g.double() - want).norm() / want.norm()) <= 1e-4
