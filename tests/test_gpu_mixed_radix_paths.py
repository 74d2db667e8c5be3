"""The unrolled mixed-radix kernels (188^2 from 512 or 640 frames of a scan on,
200^2 from 80 to 500, by the mode count) over several iterations: the update without a second read of psi, the
one that forms eps_psi, and their graph replay in a batch of scans."""
import numpy as np
import pytest

from test_gpu_batch import _torch, say, uneven_scans
from test_gpu_parity import psi_free_case

pytestmark = pytest.mark.gpu


# three iterations with and without DM_FLAG_PSI_ERROR_LAST against the oracle,
# the first and a middle mode count of a wave each, and more modes than waves;
# whole groups of eight views and remainders
@pytest.mark.parametrize("seed,n,f,m", [(401, 221, 200, 1), (402, 113, 200, 3), (403, 9, 200, 9),
                                        (404, 128, 188, 4), (405, 59, 188, 11)])
def test_psi_free_update_unrolled_kernels(seed, n, f, m):
    psi_free_case(seed, n, f, m, f + 70, f + 61, 1)


# one batch of large scans, one of a large and a small scan (both kernel sets in
# the graph): calls of 3, 2 and 1 iterations, replayed and launched eagerly
@pytest.mark.parametrize("f,m,sizes", [(200, 2, (165, 170)), (188, 2, (20, 256))])
def test_graph_replay_unrolled_kernels(f, m, sizes):
    torch = _torch()
    from paper_1808_10375_amd import dm
    scans = uneven_scans(seed=410, sizes=sizes, f=f, m=m, objs=(f + 80, f + 60))
    say(f"case graph replay F={f} M={m}, {sizes} views")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        g = dm.DMBatch(scans, flags=dm.DM_FLAG_GRAPH | dm.DM_FLAG_PSI_ERROR_LAST, stream=stream)
    e = dm.DMBatch(scans, flags=dm.DM_FLAG_PSI_ERROR_LAST)
    done = 0
    for n in (3, 2, 1):
        g.iterate(n)
        e.iterate(n)
        done += n
        stream.synchronize()
        torch.cuda.synchronize()
        for s in range(len(scans)):
            pairs = ((g.object(s), e.object(s)), (g.probe(s), e.probe(s)))
            stream.synchronize()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in pairs), (done, s)
            for x, y in zip(g.error_history(s, 1, done), e.error_history(s, 1, done)):
                assert x["eps_probe"] == y["eps_probe"] and x["eps_obj"] == y["eps_obj"]
                assert x["eps_psi"] == y["eps_psi"] or (np.isnan(x["eps_psi"])
                                                        and np.isnan(y["eps_psi"]))
    g.free()
    e.free()
