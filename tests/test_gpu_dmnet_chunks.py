"""The chunk-layout matrix-core convolutions of the warm-start network (channel
counts that are multiples of 32) on numbers whose sums are exact in float32.

Inputs are small integers and each output channel has four weights of +-1, so
every product sum of the forward pass is an integer multiple of 1/4 below
2^24 / 4 in any order: the GPU and the float64 emulation (which round the same
activations to bfloat16) have to agree to the last bit.  Where the number of
outputs is a power of two the output gradient is exact as well; the weight
gradients then sum products of bfloat16 numbers of mixed exponents, and agree
to float32 rounding (a bfloat16 rounding that falls on the other side moves a
gradient by about 1e-3, a wrong index by order one)."""
import numpy as np
import pytest
import torch

from oracle import cnn_oracle as net

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def exact_case(seed, n, size, c0, levels):
    rng = np.random.default_rng(seed)
    params = []
    for i, p in enumerate(net.init_params(seed, c0, levels)):
        if i % 2 or p.shape[2] == 1:
            params.append(rng.integers(-1, 2, p.shape).astype(np.float64))
            continue
        w = np.zeros((p.shape[0], p.shape[1] * 9))
        for row in w:
            at = rng.choice(row.size, 4, replace=False)
            row[at] = rng.choice([-1.0, 1.0], 4)
        params.append(w.reshape(p.shape))
    x = rng.integers(0, 4, (n, 1, size, size)).astype(np.float64)
    target = rng.integers(-3, 4, (n, 2, size, size)).astype(np.float64)
    return params, x, target


# one chunk and several; rows of 8 to 96 pixels (shorter than a tile, no
# multiple of it, and longer than a 64-position tile, which stages its three
# tap rows apart); several samples in a tile; channels 384 -> 128 at 32 x 32,
# which do not fit LDS together
@pytest.mark.parametrize("n,size,c0", [(1, 8, 32), (5, 12, 32), (2, 32, 32), (3, 36, 64),
                                       (1, 96, 64), (1, 32, 128), (70, 8, 64)])
def test_chunk_convolutions_exact(n, size, c0):
    from paper_1808_10375_amd import dmnet
    levels = 2
    params, x, target = exact_case(7 * n + size + c0, n, size, c0, levels)
    m = dmnet.DMNet(n + 1, size=size, base_ch=c0, levels=levels, device=DEV)
    m.set_params(net.flatten(params))
    xd = torch.as_tensor(x.astype(np.float32)).to(DEV)
    l_ref, g_ref, y_ref = net.loss_and_grads(params, x, target, levels,
                                             act_round=net.bf16_round)
    assert np.abs(y_ref).max() < 2 ** 21
    y = m.forward(xd).cpu().numpy()
    assert np.array_equal(y, y_ref.astype(np.float32))
    loss, g = m.loss_grad(xd, torch.as_tensor(target.astype(np.float32)).to(DEV))
    # float32 sums of n * 2 * size^2 squares against float64
    assert abs(loss - l_ref) <= 1e-5 * l_ref
    if (n * size * size) & (n * size * size - 1) == 0:
        g, g_ref = g.cpu().numpy().astype(np.float64), net.flatten(g_ref)
        assert np.linalg.norm(g - g_ref) <= 1e-4 * np.linalg.norm(g_ref)
