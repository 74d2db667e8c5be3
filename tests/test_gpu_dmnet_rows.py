"""3x3 convolutions of the warm-start network whose input channels do not fit
LDS together: staged tap row by tap row, all channels at once or in groups."""
import pytest
import torch

import test_gpu_dmnet_chunks as chunks
from test_gpu_dmnet_tiles import network, torch_forward

pytestmark = pytest.mark.gpu


# forward and gradients against the float64 oracle: 768 -> 256 channels (two
# groups of 15 and 9 chunks of 32; 64 channels a block), 480 -> 160 (two of 8
# and 7; 32 channels a block), and their data gradients; several samples
@pytest.mark.parametrize("n,size,c0", [(1, 16, 256), (1, 16, 160), (4, 8, 256)])
def test_wide_networks_exact(n, size, c0):
    print(f"case conv rows n={n} size={size} base={c0}", flush=True)
    chunks.test_chunk_convolutions_exact(n, size, c0)


# forward against plain torch: rows longer than a block's run of positions, no
# multiple of it, and several samples in a run; one group (384 channels) and two
@pytest.mark.parametrize("n,size,c0", [(1, 140, 128), (3, 62, 128), (2, 46, 160), (5, 20, 256)])
def test_wide_networks_forward_exact(n, size, c0):
    print(f"case conv rows forward n={n} size={size} base={c0}", flush=True)
    params, x, _ = chunks.exact_case(n + size + c0, n, size, c0, 2)
    y = network(n, size, c0, params).forward(torch.from_numpy(x).float().to(chunks.DEV)).cpu()
    assert torch.equal(y, torch_forward(params, x).float())
