"""Detection at every size class of the suppression's sort: candidate counts
at and around 0, 1, 64, 128 and 256 (in one wave's registers) and past them
(in LDS), equal scores, the kept-box cap, and class counts around the decode's
register variants.  Kept lists against the oracle, as in test_gpu_detect.py."""
import numpy as np
import pytest

from tests.test_gpu_detect import compare

pytestmark = pytest.mark.gpu

ANCHORS = range(8)  # four anchors (compare() draws them)


def _head(counts, classes, side, equal):
    """One image per entry of counts: that many boxes of class 0 with a score
    near 0.9 (or all the same), every other box and class near 0."""
    rng = np.random.default_rng([len(counts), classes, side])
    A = len(ANCHORS) // 2
    y = np.zeros((len(counts), A, 5 + classes, side, side), np.float32)
    y[:, :, :4] = rng.normal(0.0, 0.7, y[:, :, :4].shape)
    y[:, :, 4] = -12.0
    y[:, :, 5] = 12.0
    for n, c in enumerate(counts):
        pick = rng.permutation(side * side * A)[:c]
        a, i, j = pick % A, pick // A // side, pick // A % side
        y[n, a, 4, i, j] = 2.0 if equal else 2.0 + rng.permutation(c) / 64.0
    return y.reshape(len(counts), A * (5 + classes), side, side)


@pytest.mark.parametrize("equal", [False, True], ids=["distinct", "equal"])
@pytest.mark.parametrize("max_det", [7, 400])
@pytest.mark.parametrize("classes", [1, 24, 25, 97])
def test_counts_around_the_sort_sizes(classes, max_det, equal):
    from paper_1811_03882_amd import dn
    counts = [0, 1, 2, 3, 63, 64, 65, 127, 128, 129, 255, 256, 257, 400]
    y = _head(counts, classes, 10, equal)
    kept, _ = compare(dn, y, len(ANCHORS) // 2, classes, 0.5, 0.45, max_det)
    assert kept > 0
