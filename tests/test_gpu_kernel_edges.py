"""One iteration against the FP64 oracle at the sizes where the smaller
kernels of the iteration can go wrong (remainders of their batches, the last
and the first size of a split)."""
import numpy as np
import pytest

from paper_1808_10375_amd import synth
import test_gpu_bf16x3 as bf16x3
from test_gpu_parity import one_step_case, say

pytestmark = pytest.mark.gpu


# k_probe_final adds 16 chunks at a time and eight modes at a time: three chunks,
# 16, 17 and 64 chunks (as many as views up to 64); one, eight, nine and 16
# modes.  Tolerances are the one-step tests' own.
@pytest.mark.parametrize("seed,n,f,m", [(81, 3, 16, 1), (82, 16, 16, 8), (83, 17, 32, 9),
                                        (84, 64, 16, 16), (85, 130, 16, 1)])
def test_probe_division_over_chunks_and_modes(seed, n, f, m):
    say(f"case probe division seed={seed} N={n} F={f} M={m}")
    one_step_case(synth.random_case(seed, n, f, m, 2 * f + 7, 2 * f + 3, perturb=0.5))


# the fused view kernel keeps a view's operands in registers below 128^2: one
# mode (nothing transformed twice), two, three and 16 modes
@pytest.mark.parametrize("seed,n,f,m", [(121, 9, 64, 1), (122, 33, 64, 2), (123, 17, 64, 3),
                                        (124, 5, 64, 16), (125, 41, 32, 2), (126, 10, 32, 5),
                                        (127, 11, 16, 3)])
def test_fused_views_and_modes(seed, n, f, m):
    say(f"case fused views seed={seed} N={n} F={f} M={m}")
    one_step_case(synth.random_case(seed, n, f, m, 2 * f + 9, 2 * f + 4, perturb=0.5))


# the column kernel of the BF16x3 form is compiled per mode count; the counts
# the form's own tests leave out, with view counts that leave the persistent
# blocks nothing (two views: fewer frames than blocks) or an uneven share
@pytest.mark.parametrize("seed,n,m", [(91, 2, 2), (92, 41, 2), (93, 9, 4), (94, 7, 6),
                                      (95, 6, 7)])
def test_bf16x3_mode_counts(seed, n, m):
    say(f"case bf16x3 modes seed={seed} N={n} M={m}")
    bf16x3.compare(synth.random_case(seed, n, 128, m, 190, 200, perturb=0.3))


# the mixed-radix frames on both kernel sets (513 x 1 and 256 x 2 frames of 188^2
# and 13 x 7 and 8 x 13 of 200^2 run the unrolled kernels): modes shared out over
# the waves of a block (up to 8 one each; above, the column kernel takes six
# waves, the inverse row kernel eight, with the last round part empty), the
# single-mode forms, and view counts with whole groups of eight views per XCD
# map and a remainder
@pytest.mark.parametrize("seed,n,f,m", [(101, 513, 188, 1), (102, 80, 200, 1), (103, 256, 188, 2),
                                        (104, 13, 200, 7), (105, 57, 188, 9), (106, 8, 200, 13),
                                        (107, 511, 188, 1), (108, 39, 200, 2)])
def test_mixed_radix_modes_and_views(seed, n, f, m):
    say(f"case mixed radix modes seed={seed} N={n} F={f} M={m}")
    one_step_case(synth.random_case(seed, n, f, m, f + 60, f + 55, perturb=0.5))


# a checkpoint's views go in and out bit for bit: below and above the size from
# which a kernel streams them (64 MB; blocks of 1024 words of 16 bytes, the last
# one partial), and from and to addresses 8 bytes off a 16-byte boundary
@pytest.mark.parametrize("n,f,shift", [(63, 256, 0), (129, 256, 0), (238, 188, 0), (130, 256, 1)])
def test_checkpoint_views_round_trip(n, f, shift):
    import torch
    from paper_1808_10375_amd import dm
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    c = synth.random_case(111, n, f, 1, f + 9, f + 12)
    ctx = dm.DMContext(torch.from_numpy(c["I"]).to(dev), c["pos"], torch.from_numpy(c["P"]).to(dev),
                       torch.from_numpy(c["O"]).to(dev))
    flat = torch.randn(2 * (n * f * f + shift), generator=g, device=dev)
    psi = torch.view_as_complex(flat[2 * shift:].view(n, 1, f, f, 2))
    ctx.set_state(psi, torch.from_numpy(c["P"]).to(dev), torch.from_numpy(c["O"]).to(dev), 0)
    back = torch.zeros(n * f * f + shift, dtype=torch.complex64, device=dev)
    dm.dm_get_state(ctx.ctx, back[shift:])
    assert np.array_equal(back[shift:].cpu().numpy(), psi.cpu().numpy().ravel())
    assert torch.equal(ctx.state()[0], psi)
    ctx.free()
