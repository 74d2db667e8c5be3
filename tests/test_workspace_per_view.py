"""What one more view adds to the workspace below 128^2: its frames, its object
numerator and index lists; no buffer that no kernel touches."""
import pytest

from paper_1808_10375_amd import dm


@pytest.mark.parametrize("f,m", [(16, 1), (32, 3), (64, 2)])
def test_workspace_grows_by_frames_and_numerator(f, m):
    def size(n):
        return dm.dm_workspace_bytes(dm.make_desc(n, f, m, 300, 300, 0.8))

    # from 256 views on the spectra slots of the streamed path stay as they are
    grown = (size(1600) - size(600)) / 1000
    frames = (m + 1) * f * f * 8
    assert frames <= grown < frames + f * f * 2 + 256
