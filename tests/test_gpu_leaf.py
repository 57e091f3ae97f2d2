"""GPU parity of the leaf kernel (boxes over runs of 32 sorted points, half-precision matrix pre-filter, exact
re-evaluation) against the CPU oracle, bit for bit, at the sizes where it can go wrong, and against the plain walk on
coordinates that strain the pre-filter's scaling."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B
from paper_2511_10442_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run(x, rs, k, direction=None, algo=3):
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    dt = None if direction is None else torch.from_numpy(direction).to(DEV)
    idx, d2 = B.fg_query_binned(B.fg_bin_points(xt, rt, k), rt, k, direction=dt, algo=algo)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), d2.cpu().numpy().view(np.uint32)


def check(x, rs, k, direction=None):
    oi, od = oracle.knn(x, rs, k, direction=direction)
    gi, gd = run(x, rs, k, direction)
    assert np.array_equal(gi, oi) and np.array_equal(gd, od.view(np.uint32))


# list sizes and both passes of a long list; splits of one leaf less, equal and one more, empty and tiny ones; ties
@pytest.mark.parametrize("d", range(2, 11))
@pytest.mark.parametrize("k", [1, 2, 17, 18, 33, 49, 64, 65, 66, 100, 128])
def test_matches_oracle(d, k):
    sizes = [1300, 5, 0, 31, 32, 33, 63, 64, 65, 900, 1, 70]
    x, rs = W.uniform(sum(sizes), d, seed=900 + 11 * d + k, sizes=sizes)
    x[100:300] = x[100]                                      # duplicates: ties on distance 0
    x[1600:2000] = x[1600] + 0.01 * (x[1600:2000] - 0.5)     # a dense cluster among sparse points
    x = np.ascontiguousarray(x)
    check(x, rs, k)
    rng = np.random.Generator(np.random.PCG64(d * 131 + k))
    check(x, rs, k, rng.integers(0, 4, size=x.shape[0]).astype(np.int32))


# at an offset of 4096 a lone point or a set of equal ones has no extent to scale by
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 64, 65, 2048, 2049, 4097])
@pytest.mark.parametrize("d", [6, 9, 10])
@pytest.mark.parametrize("offset", [0.0, 4096.0, 1e30])
def test_small_sizes(n, d, offset):
    x, rs = W.uniform(n, d, seed=n + d)
    check(np.ascontiguousarray(x + np.float32(offset)), rs, min(20, n + 2))
    if n <= 65:
        check(np.ascontiguousarray(x + np.float32(offset)), rs, 128)


# far from the origin, tiny and huge scales, a lattice (many equal distances), one far outlier, squares that overflow
# and squares that underflow
@pytest.mark.parametrize("d", [2, 6, 10])
@pytest.mark.parametrize("kind", ["shifted", "tiny", "huge", "lattice", "outlier", "overflow", "underflow", "line"])
def test_coordinates_that_strain_the_filter(d, kind):
    x, rs = W.uniform(1500, d, seed=77 + d)
    if kind == "shifted": x = x + np.float32(1000.0)
    if kind == "tiny": x = x * np.float32(1e-12)
    if kind == "huge": x = x * np.float32(1e15)
    if kind == "lattice": x = np.floor(x * 4).astype(np.float32)
    if kind == "outlier": x[7] = 1e6
    if kind == "overflow": x = x * np.float32(1e30)
    if kind == "underflow": x = x * np.float32(1e-24)
    if kind == "line": x[:, 1:] = 0.25
    check(np.ascontiguousarray(x.astype(np.float32)), rs, 24)


# three levels of boxes (more than 131 072 points): every row against the plain walk
@pytest.mark.parametrize("d,k", [(3, 16), (6, 20)])
def test_three_levels(d, k):
    x, rs = W.uniform(140_001, d, seed=3, sizes=[100_000, 40_001])
    a, b = run(x, rs, k), run(x, rs, k, algo=1)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


# two dimensions and more than 2^22 points: the heaviest tiles are the leaf kernel's, the others the tile kernel's, in both
# passes of a long list; against the tile kernel alone on every row and the oracle on sampled ones
@pytest.mark.parametrize("k", [9, 70])
def test_dense_tiles_of_two_dimensions(k):
    rng = np.random.Generator(np.random.PCG64(41))
    n = (1 << 22) + 777
    r = rng.random(n) ** 3
    phi = rng.random(n) * 2.0 * np.pi
    x = np.ascontiguousarray(np.stack([r * np.cos(phi), r * np.sin(phi)], axis=1).astype(np.float32))
    rs = np.array([0, 2_500_000, 2_500_000, 4_000_000, n], dtype=np.int32)
    a, b = run(x, rs, k, algo=0), run(x, rs, k, algo=4)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    near = np.argsort(r)[:20]                                     # inside the densest bin
    rows = np.unique(np.concatenate([near, rng.choice(n, size=40, replace=False)])).astype(np.int64)
    oi, od = oracle.knn_rows(x, rs, k, rows)
    assert np.array_equal(a[0][rows], oi) and np.array_equal(a[1][rows], od.view(np.uint32))


# options filled with zeros, or with a hand-over rule alone, choose no kernel: the default serves the call and the tile
# kernel's rule has no effect (the scratch block counts the queries that the tile kernel hands over)
@pytest.mark.parametrize("n,d", [(2000, 3), (5000, 6)])
@pytest.mark.parametrize("defer_lanes", [0, 64])
def test_a_hand_over_rule_chooses_no_kernel(n, d, defer_lanes):
    x, rs = W.uniform(n, d, seed=5)
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    bn = B.fg_bin_points(xt, rt, 10)
    B.fg_query_binned(bn, rt, 10, algo=4, defer_lanes=64)
    handed = int(bn.work_count.item())
    idx, d2 = B.fg_query_binned(bn, rt, 10, defer_lanes=defer_lanes)
    torch.cuda.synchronize()
    assert handed > 0 and int(bn.work_count.item()) == 0
    oi, od = oracle.knn(x, rs, 10)
    assert np.array_equal(idx.cpu().numpy(), oi) and np.array_equal(d2.cpu().numpy().view(np.uint32), od.view(np.uint32))


# few points ask: whole groups of eight tiles handed to the list kernel, groups that are not, the last group short, and both
# passes of a long list
@pytest.mark.parametrize("d,k", [(3, 20), (6, 64), (6, 100), (8, 17), (10, 33)])
@pytest.mark.parametrize("share", [0.0, 0.02, 0.3, 0.5, 1.0])
def test_few_points_ask(d, k, share):
    sizes = [3000, 0, 1, 700, 1333]
    n = sum(sizes)
    x, rs = W.uniform(n, d, seed=d + k, sizes=sizes)
    rng = np.random.Generator(np.random.PCG64(k + d))
    direction = np.where(rng.random(n) < share, 3, 0).astype(np.int32)
    direction[n // 2:][rng.random(n - n // 2) < 0.8] = 1      # the second half of the rows mostly asks
    check(x, rs, k, direction)


# what sends blocks to the exact comparison: copies of few points, two tight clusters in a tile, far outliers; and tiles in
# which no, one or many steps of the sorted order stand out
@pytest.mark.parametrize("d", [2, 6, 8, 10])
@pytest.mark.parametrize("kind", ["copies", "two_clusters", "far", "one_step", "steps"])
@pytest.mark.parametrize("k", [12, 66])
def test_grain_and_groups(d, kind, k):
    rng = np.random.Generator(np.random.PCG64(d + k))
    n = 3000
    x = rng.random((n, d))
    if kind == "copies": x = x[rng.integers(0, 7, size=n)]
    if kind == "two_clusters": x = np.where(np.arange(n)[:, None] % 2, 0.1, 0.9) + 1e-5 * rng.standard_normal((n, d))
    if kind == "far": x[rng.random(n) < 0.01] *= 1e4
    if kind == "one_step": x[:, :min(d, 5)] = np.where(np.arange(n)[:, None] < n // 3, 0.25, 0.75)
    if kind == "steps": x = np.floor(x * 3) / 3 + 1e-4 * rng.random((n, d))
    check(np.ascontiguousarray(x.astype(np.float32)), np.array([0, 2100, n], dtype=np.int32), k)
