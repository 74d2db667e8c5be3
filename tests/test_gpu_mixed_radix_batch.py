"""Batches of scans with frames of 188 and 200 pixels: each scan of a batch
runs the kernels that it runs alone, those for few frames or the unrolled ones
by its own frame count, and so gives the same bits."""
import numpy as np
import pytest

from test_gpu_batch import _torch, say, single, uneven_scans

pytestmark = pytest.mark.gpu


def same(a, b):
    return a == b or (np.isnan(a) and np.isnan(b))


# (frame, modes, views of the scans): the unrolled kernels start at 512 frames
# (views x modes) at 188^2 x 2 modes, at 220 at 200^2 x 1, at 330 at 200^2 x 3, at 500
# or with 9 to 19 views at 200^2 x 9.  Scans below that count which together reach
# it; both kinds in one batch, the larger scan first; scans above it only, with
# and without whole groups of eight views.
@pytest.mark.parametrize("f,m,sizes", [(200, 1, (100, 90, 41)), (188, 2, (130, 128)),
                                       (200, 1, (225, 20, 230, 7)), (200, 3, (112, 115)),
                                       (200, 9, (11, 9))])
@pytest.mark.parametrize("last", [False, True])
def test_mixed_radix_batch_equals_each_scan_alone(f, m, sizes, last):
    _torch()
    from paper_1808_10375_amd import dm
    objs = [f + 60 + 20 * (i % 3) for i in range(len(sizes))]
    scans = uneven_scans(seed=200, sizes=sizes, f=f, m=m, objs=objs)
    say(f"case batch of {sizes} views, F={f} M={m}, eps_psi {'last' if last else 'every'}")
    flags = dm.DM_FLAG_PSI_ERROR_LAST if last else 0
    b = dm.DMBatch(scans, flags=flags)
    b.iterate(3)
    for s, sc in enumerate(scans):
        ctx = single(sc, flags=flags)
        ctx.iterate(3)
        assert np.array_equal(b.object(s).cpu().numpy(), ctx.object().cpu().numpy()), s
        assert np.array_equal(b.probe(s).cpu().numpy(), ctx.probe().cpu().numpy()), s
        for x, y in zip(b.error_history(s, 1, 3), ctx.error_history(1, 3)):
            assert all(same(x[k], y[k]) for k in ("eps_psi", "eps_obj", "eps_probe")), (s, x, y)
        ctx.free()
    b.free()
