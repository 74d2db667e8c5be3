"""Two live contexts of different mode counts.  The dynamic LDS that a kernel
may take is an attribute of the kernel, not of a context: a context of few
modes made later must not lower it for an earlier one of many."""
import ctypes

import numpy as np
import pytest

from paper_1808_10375_amd import synth
from test_gpu_batch import _torch, say, single

pytestmark = pytest.mark.gpu


def scan(seed, n, f, m):
    c = synth.random_case(seed, n, f, m, f + 40, f + 33, perturb=0.3)
    return dict(I=c["I"], pos=c["pos"], P0=c["P"], O0=c["O"], beta=c["beta"])


class FuncAttributes(ctypes.Structure):  # hipFuncAttributes
    _fields_ = [("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int),
                ("constSizeBytes", ctypes.c_size_t), ("localSizeBytes", ctypes.c_size_t),
                ("maxDynamicSharedSizeBytes", ctypes.c_int), ("rest", ctypes.c_int * 16)]


def lds_limit(kernel):
    """the dynamic LDS limit of a kernel of libdm.so, by its mangled name"""
    from paper_1808_10375_amd import dm
    a = FuncAttributes()
    at = ctypes.addressof(ctypes.c_char.in_dll(dm.lib(), kernel))
    assert dm.lib().hipFuncGetAttributes(ctypes.byref(a), ctypes.c_void_p(at)) == 0
    return a.maxDynamicSharedSizeBytes


SIG = "EEvPKNS_7ScanDevEPK15HIP_vector_typeIiLj2EEPKS4_IfLj2EEi"
KERNELS = {16: ["_ZN3dmk6k_colsILi16E" + SIG + "ii"],
           188: ["_ZN3dmk10k_mix_colsILi188ELb0E" + SIG + "i",
                 "_ZN3dmk14k_mix_rows_invILi188ELb0ELb0E" + SIG,
                 "_ZN3dmk14k_mix_rows_invILi188ELb1ELb0E" + SIG],
           200: ["_ZN3dmk10k_mix_colsILi200ELb0E" + SIG + "i",
                 "_ZN3dmk14k_mix_rows_invILi200ELb0ELb0E" + SIG,
                 "_ZN3dmk14k_mix_rows_invILi200ELb1ELb0E" + SIG]}


def state(ctx):
    return [x.cpu().numpy() for x in ctx.state()[:3]]


# kernels whose blocks take over 64 KB at the first mode count: the unrolled
# column and inverse row kernels of 188^2 and 200^2 (both contexts with frames
# enough to take them), the column kernel of the power-of-two frames (16 modes of 16^2)
@pytest.mark.parametrize("f,many,few", [(200, (10, 8), (165, 2)), (188, (40, 16), (256, 2)),
                                        (16, (9, 16), (9, 1))])
def test_older_context_of_more_modes_still_runs(f, many, few):
    _torch()
    from paper_1808_10375_amd import dm
    say(f"case LDS limit F={f}: {many} views x modes, then {few}")
    flags = dm.DM_FLAG_MULTIPASS if f <= 128 else 0
    a_scan, b_scan = scan(301, many[0], f, many[1]), scan(302, few[0], f, few[1])
    a = single(a_scan, flags=flags)
    a.iterate(2)
    want = state(a)
    a.free()
    for last in (0, dm.DM_FLAG_PSI_ERROR_LAST):
        a = single(a_scan, flags=flags | last)
        before = [lds_limit(k) for k in KERNELS[f]]
        b = single(b_scan, flags=flags | last)
        after = [lds_limit(k) for k in KERNELS[f]]
        say(f"  limits {before} -> {after}")
        assert all(y >= x for x, y in zip(before, after))
        b.iterate(2)
        a.iterate(2)
        b.iterate(2)
        got = state(a)
        if not last:
            assert all(np.array_equal(x, y) for x, y in zip(got, want))
        else:
            assert all(np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y)
                       for x, y in zip(got[:1] + got[2:], want[:1] + want[2:]))
        a.free()
        b.free()
