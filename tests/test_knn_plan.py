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
    p = hn.knn_plan(form, max(1, n // part), n, 128, 32)
    assert 1 <= p.splits <= 32 and p.split_rows % 128 == 0
    assert (p.splits - 1) * p.split_rows < n <= p.splits * p.split_rows


@pytest.mark.parametrize("form", [SPLIT, FP32])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("part", [1, 3, 10])
def test_later_forms_split_only_to_fill_the_chip(form, n, part):
    """Each split fills lists of its own: a pass with a block for every CU is
    not split, and the others to four rounds of 512 blocks at most."""
    rows = max(1, n // part)
    blocks = -(-rows // 128)
    p = hn.knn_plan(form, rows, n, 128, 32)
    assert p.splits == 1 if blocks >= 256 else p.splits * blocks <= 2048


@pytest.mark.parametrize("degree", [17, 24, 32])
@pytest.mark.parametrize("d", [8, 32, 128])
@pytest.mark.parametrize("n", [n for n in SIZES if n > 128])
def test_fp16_bound_of_more_than_16_neighbours_takes_two_splits(n, d, degree):
    """A split's lists bound a row near rank 44; with R up to 32 the proof
    needs the rank of two, whatever the number of blocks."""
    assert hn.knn_plan(HALF, n, n, d, degree).splits >= 2


@pytest.mark.parametrize("form", [HALF, SPLIT, FP32])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("d", [32, 128, 768])
def test_lists_of_a_launch_are_bounded(form, n, d):
    """512 bytes a row and split: at most 1 GiB for the largest launch, and
    the pilot's launch is no larger."""
    p = hn.knn_plan(form, n, n, d, 32)
    rows = min(n, 128 * p.slice_blocks)
    assert p.slice_blocks >= 1 and rows * p.splits <= 1 << 21
    assert p.pilot_blocks <= p.slice_blocks


@pytest.mark.parametrize("d", [16, 128, 768])
@pytest.mark.parametrize("n", [33_000, 50_000, 65_537, 100_000, 1_000_000, 10_000_000])
def test_fp16_pass_over_a_large_layer_has_a_pilot(n, d):
    """One round of blocks, at most two thirds of the layer, decides before the
    whole layer is paid for; the other forms have none."""
    p = hn.knn_plan(HALF, n, n, d, 32)
    assert 0 < p.pilot_blocks <= -(-n // 128) * 2 // 3
    assert p.pilot_blocks * p.splits <= 768
    assert hn.knn_plan(SPLIT, n, n, d, 32).pilot_blocks == 0
    assert hn.knn_plan(FP32, n, n, d, 32).pilot_blocks == 0


@pytest.mark.parametrize("n", [2_100_000, 5_000_000, 10_000_000])
def test_very_large_layers_take_no_extra_splits(n):
    """They have rounds enough: only the proof of more than 16 neighbours asks
    for a second split."""
    assert hn.knn_plan(HALF, n, n, 32, 16).splits == 1
    assert hn.knn_plan(HALF, n, n, 32, 32).splits == 2
