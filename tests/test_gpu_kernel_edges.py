"""One iteration against the FP64 oracle at the sizes where the smaller
kernels of the iteration can go wrong (remainders of their batches, the last
and the first size of a split)."""
import pytest

from paper_1808_10375_amd import synth
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
