"""Clearing on maps and at ray steps at the edges of the march's forms, alone and
in a batch, against the oracle, which tests every sample: marks, state and bound
bit for bit."""
import pytest

from test_gpu_clear_long_rays import _check
from test_gpu_clear_march import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# nx, ny, step / r, sensor (cells), reach (cells), n, valid, flat.  Maps of one row or
# column of 8 x 8 blocks, or of 32 x 32 superblocks, down to one block; the counts of
# blocks on both sides of the maxima's padding (64 to 256 bytes).
NARROW = [
    (8, 300, 1.0, (4.0, 20.0), 290, 700, 0.6, True),
    (300, 7, 1.0, (20.0, 3.0), 290, 700, 0.6, True),
    (5, 5, 1.0, (2.5, 2.5), 9, 300, 0.9, False),
    (8, 8, 0.3, (1.0, 7.0), 12, 300, 0.9, False),
    (9, 512, 1.0, (4.0, 500.0), 520, 700, 0.6, True),
    (3, 504, 1.0, (1.0, 10.0), 520, 500, 0.6, True),
    (4, 512, 1.0, (1.0, 10.0), 520, 500, 0.6, True),
    (512, 8, 0.25, (5.0, 4.0), 520, 500, 0.6, True),
    (2050, 8, 1.0, (1000.0, 4.0), 1100, 700, 0.6, True),
    (8, 2050, 1.0, (4.0, 1000.0), 1100, 50000, 0.6, True),
]


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("k", range(len(NARROW)))
def test_narrow_maps(dev, k, ub, batched):  # noqa: F811
    _check(dev, NARROW[k], 5000 + 10 * k + ub, ub, batched)
