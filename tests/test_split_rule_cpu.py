"""The split count that the library chooses for a small conv on its own, from
the scratch it asks for (host logic, no GPU).  A thread of the separate finish
reads one partial after the other, four times as many under a fused pool: on
one 8x8 image the reads of 16 splits take longer than the conv."""
import pytest

from paper_1811_03882_amd import dn


def _splits(dtype, cin, cout, side, pool):
    d = dn.conv_desc(1, side, side, cin, cout, 3, 1, 1, 1, 0.1, pool, 0, dtype)
    ws = dn.conv_sizes(d)[2]
    return max(1, ws // (side * side * dn.channel_pad(dtype, cout) * 4))


@pytest.mark.parametrize("dtype,cin", [(dn.F32, 64), (dn.BF16, 128), (dn.FP8, 256)], ids=["f32", "bf16", "fp8"])
@pytest.mark.parametrize("cout", [64, 256])
@pytest.mark.parametrize("side", [4, 8, 14])
def test_few_splits_on_small_images(dtype, cin, cout, side):
    assert _splits(dtype, cin, cout, side, 2) <= 4
    assert _splits(dtype, cin, cout, side, 0) <= 8
