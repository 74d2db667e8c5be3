"""The views of a checkpoint at the size from which a kernel copies them (64 MB),
and under stream capture."""
import pytest

from paper_1808_10375_amd import synth
from test_gpu_batch import _torch, say

pytestmark = pytest.mark.gpu


def context(n, f, stream=None):
    torch = _torch()
    from paper_1808_10375_amd import dm
    c = synth.random_case(112, n, f, 1, f + 9, f + 12)
    I, P, O = (torch.from_numpy(c[k]).to("cuda:0") for k in ("I", "P", "O"))
    torch.cuda.synchronize()
    return dm.DMContext(I, c["pos"], P, O, stream=stream), P, O


def views(n, f, seed):
    torch = _torch()
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.complex(torch.randn((n, 1, f, f), generator=g, device="cuda:0"),
                         torch.randn((n, 1, f, f), generator=g, device="cuda:0"))


# 512 KB a view: one view below 64 MB, exactly 64 MB, one above; blocks of 1024
# words of 16 bytes, the last one of 188^2 views partial
@pytest.mark.parametrize("n,f", [(127, 256), (128, 256), (129, 256), (239, 188)])
def test_views_in_and_out_at_the_copy_limit(n, f):
    torch = _torch()
    say(f"case checkpoint copy N={n} F={f}")
    ctx, P, O = context(n, f)
    psi = views(n, f, n)
    ctx.set_state(psi, P, O, 0)
    assert torch.equal(ctx.state()[0], psi)
    ctx.free()


@pytest.mark.parametrize("n", [100, 130])
def test_state_set_by_a_replayed_graph(n):
    """dm_set_state recorded into a graph and replayed three times, with other
    views in the same buffer and eager work between: below and above the limit."""
    torch = _torch()
    say(f"case checkpoint copy in a graph N={n}")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx, P, O = context(n, 256, stream)
        psi = views(n, 256, 1)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.set_state(psi, P, O, 0)
    for seed in (2, 3, 4):
        psi.copy_(views(n, 256, seed))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()
        assert torch.equal(ctx.state()[0], psi), seed
    ctx.free()
