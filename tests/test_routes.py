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
    (40_000, 8, 16, 834, "leaf"), (40_000, 8, 16, 833, "group"), (10_000, 8, 16, 1667, "leaf"), (10_000, 8, 16, 1666, "group"), (40_000, 3, 24, 8000, "group"),
    (40_000, 3, 10, 625, "group or tile"), (40_000, 3, 10, 626, "tile")])
def test_splits_of_a_few_points(n, d, k, splits, expect):
    assert served(n, d, k, splits) == expect
