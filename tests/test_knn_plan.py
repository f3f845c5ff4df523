"""How the kNN build splits and slices its Gram passes (host only)."""
import pytest

from paper_2505_17368_amd import henn as hn

HALF, SPLIT, FP32 = 0, 1, 2
SIZES = [1, 127, 129, 5000, 20_000, 50_000, 65_537, 130_000, 262_144, 500_000, 1_000_000,
         1_200_000, 10_000_000]


@pytest.mark.parametrize("form", [HALF, SPLIT, FP32])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("part", [1, 3, 10])
def test_splits_cover_the_layer(form, n, part):
    """Every split holds candidates, whole 128-candidate tiles, and together
    they are the layer."""
    p = hn.knn_plan(form, max(1, n // part), n, 128)
    assert 1 <= p.splits <= 32 and p.split_rows % 128 == 0
    assert (p.splits - 1) * p.split_rows < n <= p.splits * p.split_rows


@pytest.mark.parametrize("form", [SPLIT, FP32])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("part", [1, 3, 10])
def test_later_forms_split_only_to_fill_the_chip(form, n, part):
    """Each split fills lists of its own: a pass whose blocks fill the chip
    (512 at once) is not split, and the others not past one round."""
    rows = max(1, n // part)
    blocks = -(-rows // 128)
    p = hn.knn_plan(form, rows, n, 128)
    assert p.splits * blocks <= max(512, blocks)
