"""A launch that fails, at every place of every chain of launches: the call says so, and nothing that would have run on what that launch did not
write is launched after it."""
import pytest

from launches import launches

FG_ERR_LAUNCH = 5

CHAINS = {
    "all pairs": ("knn", 1000, 3, 1, 10, 0),
    "group kernel": ("knn", 6000, 4, 1, 20, 0),
    "group kernel, two passes": ("knn", 20000, 8, 1, 100, 0),
    "few points, votes": ("knn", 24000, 3, 4, 12, 0),
    "few tiles": ("knn", 60000, 3, 1, 16, 0),
    "tile or group kernel": ("knn", 100000, 4, 2, 40, 0),
    "tile or group kernel, two passes": ("knn", 100000, 3, 1, 100, 0),
    "ranked": ("knn", 1000000, 3, 10, 32, 0),
    "ordered, leaf and tile kernel": ("knn", 1200000, 2, 5, 16, 0),
    "ordered, two passes": ("knn", 1200000, 2, 5, 80, 0),
    "leaf kernel": ("knn", 200000, 8, 1, 64, 0),
    "leaf kernel, two passes": ("knn", 300000, 6, 1, 70, 0),
    "leaf kernel, direction flags": ("knn", 200000, 6, 1, 70, 1),
    "tile kernel, direction flags": ("knn", 100000, 4, 2, 40, 1),
    "counted": ("counted", 100000, 3, 1, 20, 0),
    "backward, binned": ("bwd", 20000, 3, 1, 16, 1),
    "backward, plain": ("bwd", 20000, 3, 1, 16, 0),
    "index matrices": ("oc", 20000, 0, 2, 16, 1),
    "index matrices without scratch": ("oc", 20000, 0, 2, 16, 0),
}

@pytest.fixture(scope="module")
def answers():
    return dict(zip(CHAINS, launches(list(CHAINS.values()), every_failure=True)))


@pytest.mark.parametrize("name", list(CHAINS))
def test_first_error_ends_the_chain(answers, name):
    status, names, rows = answers[name]
    assert status == 0 and len(names) >= 1 and len(rows) == len(names)
    for fail, status, made in rows:
        assert status == FG_ERR_LAUNCH and made == fail, "launch %d of %d failed: status %d, %d launches" % (fail, len(names), status, made)
