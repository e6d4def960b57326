"""A mixer workspace sized for a batch serves every smaller batch
(dmpt_mixer_workspace_bytes: scratch for batches of up to `batch` states), on
both sides of the batches where the number of workgroups changes.  No GPU."""
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2409_17033_amd", "libdmpt.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libdmpt.so not built")


@pytest.mark.parametrize("n", [1, 16, 32, 64, 65, 128, 1000, 2048, 16384, 65536])
@pytest.mark.parametrize("w,h", [(0, 1), (4, 40), (32, 256), (64, 256), (70, 64), (8, 300)])
def test_workspace_grows_with_the_batch(n, w, h):
    from paper_2409_17033_amd._lib import load
    size = load().dmpt_mixer_workspace_bytes
    last = 0
    for b in [1, 2, 3, 5, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 85, 86, 127, 128, 129, 130, 171, 200, 255, 256, 257,
              258, 300, 511, 512, 513, 600, 1024, 1025, 4096]:
        if b * n > 1 << 20 or b * n * (4 * w + 3 + 2 * h) > 1 << 31:
            break
        got = size(n, w, h, b)
        assert got > 0 and got >= last, (b, got, last)
        last = got
