"""Inputs on which the default choice of kernels was once much slower than another kernel of the library on the same call:
both are timed in turn on the same inputs, the shortest of several runs each, and the bound lies between the ratio that
was wrong and the one that is right."""
import numpy as np
import pytest
import torch

from paper_2511_10442_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def shortest(calls, runs=7, reps=3):
    """Microseconds of each call, in turn."""
    best = [float("inf")] * len(calls)
    for _ in range(runs + 1):                            # the first run warms up
        for i, call in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(reps):
                call()
            b.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) / reps * 1e3)
    print("us:", ["%.1f" % b for b in best])
    return best


def cloud(kind, n, d):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(17)
    x = torch.rand(n, d, generator=gen, device=DEV)
    pick = lambda m: torch.randint(0, m, (n,), generator=gen, device=DEV)
    if kind == "lattice":
        return torch.floor(x * 4)
    if kind.startswith("clusters"):
        count, width = {"clusters_fine": (5000, 0.01), "clusters_tight": (50, 0.001)}[kind]
        return x[:count][pick(count)] + width * torch.randn(n, d, generator=gen, device=DEV)
    if kind == "outliers":
        x[torch.rand(n, generator=gen, device=DEV) < 0.001] *= 1000.0
    return x


# the default from six dimensions on against the tile kernel (query stage alone)
@pytest.mark.parametrize("kind,n,d,k,bound", [
    ("lattice", 200_000, 6, 16, 2.0),                    # tiles that wrap: 5.5, now 1.1
    ("clusters_fine", 1_000_000, 6, 16, 1.5),            # 2.3, now 1.1
    ("clusters_tight", 200_000, 8, 64, 1.6),             # tiles over two clusters: 2.0, now 1.3
    ("outliers", 60_000, 10, 64, 0.65),                  # 0.8, now 0.48
])
def test_leaf_kernel_against_tile_kernel(kind, n, d, k, bound):
    x = cloud(kind, n, d).contiguous()
    rs = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(x, rs, k)
    out = [(torch.empty((n, k), dtype=torch.int32, device=DEV), torch.empty((n, k), device=DEV)) for _ in range(2)]
    t = shortest([lambda: B.fg_query_binned(bn, rs, k, *out[0]), lambda: B.fg_query_binned(bn, rs, k, *out[1], algo=4)])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert t[0] <= bound * t[1], "%s: %.0f against %.0f us" % (kind, t[0], t[1])


# two dimensions, a million points of strongly varying density: dense tiles by the leaf kernel against the tile kernel alone
# (1.0 while the choice began at four million points, now 0.5)
def test_dense_tiles_below_four_million_points():
    gen = torch.Generator(device=DEV)
    gen.manual_seed(17)
    n, k = 1_200_000, 16
    rand = lambda *shape: torch.rand(*shape, generator=gen, device=DEV, dtype=torch.float64)
    r, phi = rand(n) ** 3, rand(n) * 6.283185307179586
    hot = (rand(1000, 2) * 2.0 - 1.0)[torch.randint(0, 1000, (n,), generator=gen, device=DEV)]
    hot = hot + 1e-3 * torch.randn(n, 2, generator=gen, device=DEV, dtype=torch.float64)
    x = torch.where(rand(n, 1) < 0.4, hot, torch.stack([r * torch.cos(phi), r * torch.sin(phi)], dim=1)).float().contiguous()
    rs = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    bn = B.fg_bin_points(x, rs, k)
    out = [(torch.empty((n, k), dtype=torch.int32, device=DEV), torch.empty((n, k), device=DEV)) for _ in range(2)]
    t = shortest([lambda: B.fg_query_binned(bn, rs, k, *out[0]), lambda: B.fg_query_binned(bn, rs, k, *out[1], algo=4)])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert t[0] <= 0.85 * t[1], "%.0f against %.0f us" % (t[0], t[1])


# with direction flags and one point in ten asking, the same
@pytest.mark.parametrize("n,d,k", [(200_000, 6, 64), (200_000, 8, 16)])
def test_few_points_ask(n, d, k):
    x = cloud("uniform", n, d)
    rs = torch.tensor([0, n], dtype=torch.int32, device=DEV)
    flags = torch.where(torch.arange(n, device=DEV) % 10 == 3, 3, 0).int()
    bn = B.fg_bin_points(x, rs, k)
    out = [(torch.empty((n, k), dtype=torch.int32, device=DEV), torch.empty((n, k), device=DEV)) for _ in range(2)]
    t = shortest([lambda: B.fg_query_binned(bn, rs, k, *out[0], direction=flags),
                  lambda: B.fg_query_binned(bn, rs, k, *out[1], direction=flags, algo=4)])
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert t[0] <= 1.0 * t[1], "%.0f against %.0f us" % (t[0], t[1])          # 1.7, now 0.4 and 0.6


# the object-condensation matrices: M and M_not together against M alone, and against the same call with rows of M for every
# member
def objects(splits, size, count, sort=False):
    rng = np.random.Generator(np.random.PCG64(splits * 7 + count))
    label, unique, unique_rs = [], [], []
    for s in range(splits):
        points = np.sort(rng.choice(size, count, replace=False)) + s * size
        weight = rng.random(count) ** 3 + 1e-3
        a = points[np.minimum(np.searchsorted(np.cumsum(weight / weight.sum()), rng.random(size)), count - 1)]
        if sort:
            a = np.sort(a)
        a[rng.random(size) < 0.1] = -1
        label.append(a)
        unique.append(points)
        unique_rs.append(np.full(count, s))
    label, unique, unique_rs = (np.concatenate(v).astype(np.int32) for v in (label, unique, unique_rs))
    members = np.bincount(label[label >= 0], minlength=splits * size)[unique]
    rs = (np.arange(splits + 1) * size).astype(np.int32)
    return [torch.from_numpy(v).to(DEV) for v in (label, unique, unique_rs, rs)], int(members.max()), int(np.median(members))


@pytest.mark.parametrize("splits,size,count,sort,clip,bound", [
    (64, 1500, 8, False, False, 4.0),                    # few objects a split: 55, now 1.5
    (10, 100_000, 50, True, False, 15.0),                # members of an object one after the other: 81, now 6.4
    (10, 100_000, 200, False, True, 2.5),                # half of the objects with more members than rows in M: 4.9, now 1.6
])
def test_rows_of_others(splits, size, count, sort, clip, bound):
    arrays, most, median = objects(splits, size, count, sort)
    u = arrays[1].numel()
    M = torch.empty((most, u), dtype=torch.int32, device=DEV)
    M_not = torch.empty((size, u), dtype=torch.int32, device=DEV)
    ws = torch.empty(max(256, B.fg_oc_helper_workspace_size(u, size)), dtype=torch.uint8, device=DEV)
    call = lambda rows, others: lambda: B.fg_oc_helper(*arrays, rows, size, others, 1, M[:rows], M_not, ws)
    t = shortest([call(median if clip else most, True), call(most, clip)])
    assert t[0] <= bound * t[1], "%.0f against %.0f us" % (t[0], t[1])


# row splits of one point, as many bounding boxes as points, against splits of five (2.9 times as long, now 1.7)
def test_bounding_boxes_of_tiny_splits():
    x = cloud("uniform", 500_000, 3)
    one = torch.arange(500_001, dtype=torch.int32, device=DEV)
    five = torch.arange(0, 500_001, 5, dtype=torch.int32, device=DEV)
    ws = torch.empty(max(B.fg_workspace_size(500_000, 3, s, 8) for s in (500_000, 100_000)), dtype=torch.uint8, device=DEV)
    t = shortest([lambda: B.fg_bin_points(x, one, 8, workspace=ws), lambda: B.fg_bin_points(x, five, 8, workspace=ws)])
    assert t[0] <= 2.3 * t[1], "%.0f against %.0f us" % (t[0], t[1])
