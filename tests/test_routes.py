"""Which kernels serve a call by default: the rules of the dispatch on both sides of their lines, from the launches that the host makes."""
import pytest

from launches import launches

SERVE = {"k_query_small": "all pairs", "k_query_group": "group", "k_query_tile_sorted": "tile", "k_query_leaf": "leaf"}


def served(n, d, k, splits=1, flags=0):
    """The kernels that may serve the call, and whether the tiles' work is estimated to choose between them."""
    status, names, _ = launches([("knn", n, d, splits, k, flags)])[0]
    assert status == 0
    return " or ".join(v for key, v in SERVE.items() if key in names)


# splits of a few points are not the group kernel's: up to five dimensions, K < 24, where the automatic grid has one bin (and, from four on, the lists fill), beyond up to 48 points
@pytest.mark.parametrize("n,d,k,splits,expect", [
    (15_000, 2, 16, 722, "tile"), (15_000, 2, 16, 721, "group"), (12_288, 2, 16, 873, "tile"), (12_288, 2, 16, 872, "group"), (12_288, 2, 20, 873, "group"),
    (15_000, 2, 20, 1000, "group"), (15_000, 3, 20, 1000, "tile"), (20_000, 3, 10, 10_000, "tile"), (20_000, 3, 10, 1539, "tile"), (20_000, 3, 10, 1538, "group"), (20_000, 3, 8, 2272, "group"),
    (20_000, 3, 8, 2273, "tile"), (20_480, 4, 16, 1281, "group"), (20_480, 4, 16, 1280, "tile"), (20_480, 4, 16, 820, "group"), (20_481, 4, 16, 1281, "tile"),
    (40_000, 5, 16, 2501, "group"), (40_000, 5, 16, 2500, "tile"), (40_000, 5, 16, 1025, "tile"), (40_000, 5, 16, 1024, "group"),
    (40_000, 8, 16, 834, "leaf"), (40_000, 8, 16, 833, "group or leaf"), (29_999, 8, 16, 625, "leaf"), (29_999, 8, 16, 624, "group"), (10_000, 8, 16, 1667, "leaf"), (10_000, 8, 16, 1666, "group"), (20_000, 3, 24, 4000, "group"),
    (40_000, 3, 10, 625, "group or tile"), (40_000, 3, 10, 626, "tile")])
def test_splits_of_a_few_points(n, d, k, splits, expect):
    assert served(n, d, k, splits) == expect


# the group kernel's lines, the votes (group or tile) beyond, the tile kernel's sizes, and the ranked ones
@pytest.mark.parametrize("n,d,k,splits,expect", [
    (4096, 3, 65, 1, "all pairs"), (4096, 3, 66, 1, "group"), (4097, 3, 8, 1, "group"), (16_384, 2, 23, 1, "group"), (16_385, 2, 23, 1, "group or tile"),
    (32_768, 2, 23, 1, "group or tile"), (32_769, 2, 23, 1, "tile"), (28_000, 2, 32, 1, "group"), (28_001, 2, 32, 1, "group or tile"), (32_768, 2, 36, 1, "group"),
    (32_769, 2, 36, 1, "tile"), (20_480, 3, 23, 1, "group"), (20_481, 3, 23, 1, "group or tile"), (29_789, 3, 23, 1, "group or tile"), (29_790, 3, 23, 1, "tile"),
    (25_000, 3, 35, 1, "group"), (25_001, 3, 35, 1, "group or tile"), (40_960, 3, 35, 1, "group or tile"), (40_961, 3, 35, 1, "tile"),
    (35_000, 3, 65, 1, "group"), (35_001, 3, 65, 1, "group or tile"), (40_960, 3, 66, 1, "group"), (40_961, 3, 66, 1, "tile"),
    (40_960, 4, 8, 1, "group"), (40_961, 4, 8, 1, "tile"), (37_500, 4, 24, 1, "group"), (37_501, 4, 24, 1, "group or tile"), (40_960, 4, 40, 1, "group"),
    (81_920, 4, 24, 5, "group"), (81_921, 4, 24, 6, "group or tile"), (72_000, 5, 24, 1, "group"), (72_001, 5, 24, 1, "group or tile"), (80_000, 5, 23, 1, "group"), (80_001, 5, 23, 1, "group or tile"),
    (76_000, 5, 65, 1, "group"), (84_000, 5, 66, 1, "group"), (84_001, 5, 66, 1, "group or tile"), (180_224, 5, 10, 11, "group"), (180_225, 5, 10, 12, "group or tile"),
    (1 << 20, 2, 16, 1, "group or tile"), (131_073, 3, 16, 1, "tile"),
    ((1 << 20) + 1, 2, 16, 1, "tile or leaf"), (44_000, 6, 35, 1, "group"), (44_001, 6, 35, 1, "group or leaf"), (56_000, 6, 17, 1, "group"), (56_001, 6, 17, 1, "group or leaf"), (61_440, 6, 36, 1, "group"), (61_441, 6, 36, 1, "leaf"),
    (44_001, 6, 17, 2, "group or leaf"), (57_000, 6, 36, 2, "group"), (57_001, 6, 36, 2, "group or leaf"), (61_440, 7, 100, 1, "group or leaf"), (61_441, 7, 100, 2, "leaf"), (42_001, 7, 10, 4, "group or leaf"),
    (48_000, 7, 10, 1, "group"), (30_000, 8, 20, 1, "group"), (30_001, 8, 20, 1, "group or leaf"), (42_000, 8, 40, 16, "group"), (49_152, 8, 40, 16, "group or leaf"), (26_001, 9, 20, 1, "group or leaf"),
    (36_864, 9, 36, 12, "group"), (36_864, 9, 36, 11, "group or leaf"), (36_865, 9, 36, 12, "leaf"), (20_000, 10, 20, 1, "group"), (28_672, 10, 20, 1, "group or leaf"),
    (28_673, 10, 10, 1, "leaf")])
def test_lines_in_the_number_of_points(n, d, k, splits, expect):
    assert served(n, d, k, splits) == expect


# with direction flags, from six dimensions on, the share that asks decides, too: below the lines as well
@pytest.mark.parametrize("n,d,k,splits,expect", [(20_000, 6, 20, 1, "group"), (20_001, 6, 20, 1, "group or leaf"), (61_440, 6, 40, 1, "group or leaf"), (61_441, 6, 40, 1, "leaf"),
                                                  (28_672, 10, 40, 12, "group or leaf"), (30_000, 6, 16, 625, "leaf"), (40_000, 5, 20, 1, "group")])
def test_direction_flags(n, d, k, splits, expect):
    assert served(n, d, k, splits, 1) == expect
