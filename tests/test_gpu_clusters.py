"""More than 16,384 points, up to five dimensions: whether the tile kernel or the group kernel serves a call is decided on the device from
the tiles' work estimates.  Both outcomes, with their passes and flags, against the two kernels asked for by name."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def cloud(kind, n, d):
    rng = np.random.Generator(np.random.PCG64(n + d))
    x = rng.random((n, d))
    if kind == "clusters": x = x[:40][rng.integers(0, 40, size=n)] + 0.01 * rng.standard_normal((n, d))
    if kind == "hits": x[: n * 9 // 10] = x[:40][rng.integers(0, 40, size=n * 9 // 10)] + 0.01 * rng.standard_normal((n * 9 // 10, d))
    if kind == "spot": x[: n // 50] = 0.3 + 0.004 * x[: n // 50]
    if kind == "copies": x = x[rng.integers(0, n // 300, size=n)]
    return np.ascontiguousarray(x[rng.permutation(n)].astype(np.float32))


# sizes that are not ranked, with votes (the smallest and the largest of them, too) and without, the smallest that is ranked and one above the last full
# tile; both passes of a long list; the largest size with a choice in three dimensions and the first beyond it
@pytest.mark.parametrize("kind", ["uniform", "clusters", "spot", "copies"])
@pytest.mark.parametrize("n,d,k", [(16_385, 2, 12), (20_500, 3, 10), (41_000, 3, 100), (44_000, 3, 70), (49_152, 2, 20), (49_153, 2, 20), (65_537, 2, 9), (65_600, 3, 100), (70_001, 4, 65), (81_920, 4, 24), (100_003, 5, 20), (1 << 17, 3, 16), ((1 << 17) + 1, 3, 16)])
def test_either_kernel(kind, n, d, k):
    x = cloud(kind, n, d)
    rs = np.array([0, n // 3, n // 3, n // 3 + 7, n], dtype=np.int32)
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    bn = B.fg_bin_points(xt, rt, k)
    ref = B.fg_query_binned(bn, rt, k, algo=4 if kind != "copies" else 5)
    for _ in range(3):                                    # the counters of one call are cleared for the next
        got = B.fg_query_binned(bn, rt, k)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    flags = torch.from_numpy(np.random.Generator(np.random.PCG64(k)).integers(0, 4, size=n).astype(np.int32)).to(DEV)
    ref = B.fg_query_binned(bn, rt, k, direction=flags, algo=5)
    got = B.fg_query_binned(bn, rt, k, direction=flags)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    got = B.fg_query_binned(bn, rt, k)
    rows = np.linspace(0, n - 1, 25).astype(np.int64)
    oi, od = oracle.knn_rows(x, rs, k, rows)
    assert np.array_equal(got[0].cpu().numpy()[rows], oi) and np.array_equal(got[1].cpu().numpy()[rows].view(np.uint32), od.view(np.uint32))


# six dimensions and more: leaf or group kernel by the crowd that the binning counts and by tiles across splits; both passes of a long list, flags
@pytest.mark.parametrize("kind", ["uniform", "clusters", "copies"])
@pytest.mark.parametrize("n,d,k,cuts", [(20_001, 6, 70, [64, 128]), (30_000, 10, 30, [5]), (44_001, 6, 20, []), (61_440, 6, 100, [30_720]), (61_440, 6, 12, [30_721]), (49_152, 8, 40, list(range(3072, 49_152, 3072))), (36_864, 9, 66, [0, 36_864]),
                                         (28_672, 10, 10, [100, 200]), (43_000, 8, 10, list(range(1000, 43_000, 1000)))])
def test_leaf_or_group_kernel(kind, n, d, k, cuts):
    x = cloud(kind, n, d)
    rs = np.array([0] + cuts + [n], dtype=np.int32)
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    bn = B.fg_bin_points(xt, rt, k)
    flags = torch.from_numpy(np.random.Generator(np.random.PCG64(k)).integers(0, 4, size=n).astype(np.int32)).to(DEV)
    for direction in (None, flags, torch.where(torch.arange(n, device=DEV) % 37 == 5, 3, 0).int()):
        ref = B.fg_query_binned(bn, rt, k, direction=direction, algo=3 if kind != "copies" else 5)
        for _ in range(2):
            got = B.fg_query_binned(bn, rt, k, direction=direction)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    whole = B.fg_binned_select_knn(xt, rt, k)
    rows = np.linspace(0, n - 1, 12).astype(np.int64)
    oi, od = oracle.knn_rows(x, rs, k, rows)
    assert np.array_equal(whole[0].cpu().numpy()[rows], oi) and np.array_equal(whole[1].cpu().numpy()[rows].view(np.uint32), od.view(np.uint32))


# Which kernel it was: the group kernel hands no query to the list kernel, the tile kernel does on both clouds (of the scattered points among
# the clusters).  Votes (below 65,537 points) and ranked tiles; both passes of a long list
@pytest.mark.parametrize("n,d,k", [(24_000, 3, 12), (70_001, 3, 100), (70_001, 4, 24), (100_003, 5, 20), (100_003, 4, 90)])
@pytest.mark.parametrize("kind", ["uniform", "hits"])
def test_the_choice(kind, n, d, k):
    xt = torch.from_numpy(cloud(kind, n, d)).to(DEV)
    rt = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(xt, rt, k)
    handed = []
    for algo in (4, 0, 4, 0):
        B.fg_query_binned(bn, rt, k, algo=algo)
        handed.append(int(bn.work_count.item()))
    assert handed[0] > 0 and handed[2:] == handed[:2]
    assert (handed[1] == 0) == (kind == "hits"), handed


# six dimensions and more: with direction flags the leaf kernel hands over tiles of which few ask, the group kernel none
@pytest.mark.parametrize("n,d,k", [(44_001, 6, 20), (61_440, 7, 20), (36_000, 8, 70), (28_672, 10, 12)])
@pytest.mark.parametrize("kind", ["uniform", "clusters"])
def test_the_choice_with_flags(kind, n, d, k):
    xt = torch.from_numpy(cloud(kind, n, d)).to(DEV)
    rt = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(xt, rt, k)
    few = torch.where(torch.arange(n, device=DEV) % 37 == 5, 3, 0).int()
    B.fg_query_binned(bn, rt, k, direction=few, algo=3)
    assert int(bn.work_count.item()) > 0
    B.fg_query_binned(bn, rt, k, direction=few)
    assert (int(bn.work_count.item()) == 0) == (kind == "clusters")


# below the lines the flags decide: half of the points ask, or few are neighbours, and the call is the group kernel's
@pytest.mark.parametrize("n,d,k", [(20_001, 6, 20), (40_000, 6, 70), (30_000, 8, 20)])
@pytest.mark.parametrize("few,rest,group", [(3, 0, False), (1, 2, True), (3, 2, True), (0, 3, True)])
def test_the_choice_by_flags(n, d, k, few, rest, group):
    xt = torch.from_numpy(cloud("uniform", n, d)).to(DEV)
    rt = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(xt, rt, k)
    flags = torch.where(torch.arange(n, device=DEV) % 37 == 5, few, rest).int()
    ref = B.fg_query_binned(bn, rt, k, direction=flags, algo=3)
    got = B.fg_query_binned(bn, rt, k, direction=flags)
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    assert (int(bn.work_count.item()) == 0) == group


# clusters, on which the tile kernel alone takes 2 to 6 times as long; uniform points, on which the group kernel takes twice as long
@pytest.mark.parametrize("kind,n,d,k", [("clusters", 100_000, 4, 20), ("clusters", 100_000, 5, 20), ("uniform", 100_000, 3, 20), ("uniform", 100_000, 2, 20),
                                          ("clusters", 24_000, 3, 12)])
def test_takes_the_faster_one(kind, n, d, k):
    xt = torch.from_numpy(cloud(kind, n, d)).to(DEV)
    rt = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(xt, rt, k)
    idx, d2 = torch.empty((n, k), dtype=torch.int32, device=DEV), torch.empty((n, k), device=DEV)
    best = {a: float("inf") for a in (0, 4, 5)}
    for _ in range(8):
        for a in best:
            p, q = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            p.record()
            B.fg_query_binned(bn, rt, k, idx, d2, algo=a)
            q.record()
            torch.cuda.synchronize()
            best[a] = min(best[a], p.elapsed_time(q))
    assert best[0] <= 1.4 * min(best[4], best[5]), best


# a captured graph of the whole call: every replay against the eager result, with eager work between
def test_captured():
    n, k = 70_000, 12
    xt = torch.from_numpy(cloud("clusters", n, 4)).to(DEV)
    rt = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    ws = B.alloc_workspace(n, 4, 1, k)
    idx, d2 = torch.empty((n, k), dtype=torch.int32, device=DEV), torch.empty((n, k), device=DEV)
    ref = [t.clone() for t in B.fg_binned_select_knn(xt, rt, k, workspace=ws, out_idx=idx, out_d2=d2)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.fg_binned_select_knn(xt, rt, k, workspace=ws, out_idx=idx, out_d2=d2)
    for _ in range(3):
        idx.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(idx, ref[0]) and torch.equal(d2, ref[1])
        got = B.fg_binned_select_knn(xt, rt, k, workspace=ws)
        assert torch.equal(got[0], ref[0])


# a call that ended before its last kernels leaves its counts of tiles behind (here: put there): the next one on the binning does not take
# places from them, and the one after that is as fast as ever
@pytest.mark.parametrize("kind,n,d,k", [("uniform", 70_001, 3, 12), ("clusters", 100_003, 4, 20), ("uniform", 70_001, 3, 80), ("clusters", (1 << 20) + 77, 2, 10),
                                          ("uniform", 70_001, 6, 12), ("clusters", 24_000, 3, 12)])
def test_counts_left_behind(kind, n, d, k):
    xt = torch.from_numpy(cloud(kind, n, d)).to(DEV)
    rt = torch.tensor([0, n // 3, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(xt, rt, k)
    algo = 4 if d == 6 else 0
    ref = [t.clone() for t in B.fg_query_binned(bn, rt, k, algo=algo)]
    tiles = (n + 63) // 64
    at = bn.raw.scratch - bn.workspace.data_ptr() + 256 + (4 * n + 255) // 256 * 256 + 8 * tiles     # class counts, then cursors
    counters = bn.workspace[at:at + 512].view(torch.int32)
    torch.cuda.synchronize()
    assert not counters.any()
    classes = bn.workspace[at - 4 * tiles:at].view(torch.int32) & 63
    for left in (torch.bincount(classes.long(), minlength=64)[:64], torch.full((64,), tiles, device=DEV), torch.eye(64, device=DEV)[9]):
        counters[:64] = left.int()
        counters[64:] = left.int()
        got = B.fg_query_binned(bn, rt, k, algo=algo)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
        assert not counters.any()
        got = B.fg_query_binned(bn, rt, k, algo=algo)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
