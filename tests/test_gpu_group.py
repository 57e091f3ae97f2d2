"""GPU parity of the group kernel (one wavefront for two or four queries, boxes over runs of 64 sorted points) against the CPU
oracle, bit for bit, at the sizes where it can go wrong."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B
from paper_2511_10442_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run(x, rs, k, direction=None, algo=5, **bins):
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    dt = None if direction is None else torch.from_numpy(direction).to(DEV)
    idx, d2 = B.fg_query_binned(B.fg_bin_points(xt, rt, k, **bins), rt, k, direction=dt, algo=algo)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), d2.cpu().numpy().view(np.uint32)


def check(x, rs, k, direction=None, **bins):
    oi, od = oracle.knn(x, rs, k, direction=direction)
    gi, gd = run(x, rs, k, direction, **bins)
    assert np.array_equal(gi, oi) and np.array_equal(gd, od.view(np.uint32))


# list sizes and both passes of a long list; splits that end inside a group of queries and inside a leaf, empty ones, ones of
# fewer points than neighbours; ties; a dense cluster
@pytest.mark.parametrize("d", range(2, 11))
@pytest.mark.parametrize("k", [1, 2, 32, 33, 34, 64, 65, 66, 100, 128])
def test_matches_oracle(d, k):
    sizes = [1300, 5, 0, 63, 64, 65, 1, 2, 3, 900, 0, 70, 127]
    x, rs = W.uniform(sum(sizes), d, seed=700 + 11 * d + k, sizes=sizes)
    x[100:300] = x[100]
    x[1700:2100] = x[1700] + 0.01 * (x[1700:2100] - 0.5)
    x = np.ascontiguousarray(x)
    check(x, rs, k)
    rng = np.random.Generator(np.random.PCG64(d * 131 + k))
    check(x, rs, k, rng.integers(0, 4, size=x.shape[0]).astype(np.int32))


# one point to several nodes of 4096; more and fewer points than neighbours; two and four queries a wavefront
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 4095, 4097, 8193, 16385])
@pytest.mark.parametrize("d", [2, 3, 6, 7])
@pytest.mark.parametrize("offset", [0.0, 4096.0])
def test_sizes(n, d, offset):
    x, rs = W.uniform(n, d, seed=n + d)
    check(np.ascontiguousarray(x + np.float32(offset)), rs, 20)


# scales at which squares overflow, underflow or lose their accuracy, lattices and copies (equal distances across the k-th
# place), a far outlier, a line, few and many bins
@pytest.mark.parametrize("d", [2, 5, 10])
@pytest.mark.parametrize("kind", ["tiny", "huge", "overflow", "underflow", "lattice", "copies", "same", "outlier", "line"])
@pytest.mark.parametrize("bins", [{}, {"n_bins": 1, "d_bin": 2}, {"n_bins": 40, "d_bin": 2}])
def test_coordinates(d, kind, bins):
    rng = np.random.Generator(np.random.PCG64(d))
    x, rs = W.uniform(2500, d, seed=77 + d)
    if kind == "tiny": x = x * np.float32(1e-12)
    if kind == "huge": x = x * np.float32(1e15)
    if kind == "overflow": x = x * np.float32(1e30)
    if kind == "underflow": x = x * np.float32(1e-24)
    if kind == "lattice": x = np.floor(x * 4)
    if kind == "copies": x = x[rng.integers(0, 9, size=2500)]
    if kind == "same": x[:] = x[0]
    if kind == "outlier": x[7] = 1e6
    if kind == "line": x[:, 1:] = 0.25
    check(np.ascontiguousarray(x.astype(np.float32)), rs, 24, **bins)


# many row splits: the search among their boundaries takes 64 at a time
@pytest.mark.parametrize("splits", [63, 64, 65, 200, 5000])
def test_many_splits(splits):
    rng = np.random.Generator(np.random.PCG64(splits))
    sizes = rng.integers(0, 4, size=splits)
    sizes[rng.integers(0, splits, size=3)] += 400
    x, rs = W.uniform(int(sizes.sum()), 3, seed=splits, sizes=sizes.tolist())
    check(x, rs, 12)


# the default takes it up to a line in n: the last size on this side, the first on the other, through the entry points that
# take it, the first against the kernels of the second
@pytest.mark.parametrize("d,k,splits,line", [(2, 10, 1, 16384), (3, 24, 1, 40960), (4, 10, 4, 40960), (4, 10, 5, 81920), (6, 70, 3, 61440), (10, 12, 1, 28672), (2, 32, 1, 28000), (3, 32, 1, 25000), (3, 65, 1, 35000), (4, 30, 2, 37500), (5, 20, 1, 80000), (5, 70, 1, 84000)])
def test_default_on_both_sides_of_the_line(d, k, splits, line):
    for n in (line, line + 1):
        x, rs = W.uniform(n, d, seed=n, sizes=[n // splits] * (splits - 1) + [n - n // splits * (splits - 1)])
        xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
        bn = B.fg_bin_points(xt, rt, k)
        ref = B.fg_query_binned(bn, rt, k, algo=4 if d < 6 else 3)
        for idx, d2 in (B.fg_query_binned(bn, rt, k), B.fg_binned_select_knn(xt, rt, k)):
            assert torch.equal(idx, ref[0]) and torch.equal(d2, ref[1])
        rows = np.linspace(0, n - 1, 40).astype(np.int64)
        oi, od = oracle.knn_rows(x, rs, k, rows)
        assert np.array_equal(ref[0].cpu().numpy()[rows], oi) and np.array_equal(ref[1].cpu().numpy()[rows].view(np.uint32), od.view(np.uint32))


# few, half and nearly all of the points ask, in runs and scattered; lists of one and two passes; tiles and splits that end anywhere
@pytest.mark.parametrize("d", [2, 5, 6, 7, 10])
@pytest.mark.parametrize("k", [1, 12, 65, 90])
@pytest.mark.parametrize("share", [0.0, 0.01, 0.1, 0.5, 0.97, "runs"])
def test_points_that_ask(d, k, share):
    sizes = [1300, 5, 0, 63, 64, 65, 1, 900, 127, 2500]
    n = sum(sizes)
    x, rs = W.uniform(n, d, seed=900 + d + k, sizes=sizes)
    rng = np.random.Generator(np.random.PCG64(d * 131 + k))
    asks = (np.argsort(x[:, 0]) % 300 < 40) if share == "runs" else rng.random(n) < share
    check(x, rs, k, np.where(asks, rng.choice([1, 3], size=n), rng.choice([0, 2], size=n)).astype(np.int32))


# splits of a few points: the kernel for 64 queries serves them up to a grid of one bin (up to five dimensions), of up to 48 points (beyond)
@pytest.mark.parametrize("n,d,k,per", [(15_000, 2, 16, 14), (15_000, 2, 16, 15), (20_000, 3, 10, 1), (20_000, 3, 10, 2), (20_000, 3, 10, 11), (20_000, 3, 10, 13), (20_000, 3, 10, 14), (10_000, 8, 16, 6), (10_000, 8, 16, 7),
                                        (40_000, 4, 8, 12), (40_000, 4, 8, 13), (40_000, 5, 16, 15), (40_000, 5, 16, 20), (40_000, 5, 16, 40), (40_000, 8, 16, 2),
                                        (40_000, 8, 16, 48), (40_000, 8, 16, 49), (40_000, 3, 10, 63), (40_000, 3, 10, 64), (30_000, 6, 24, 5)])
def test_splits_of_a_few_points(n, d, k, per):
    x, _ = W.uniform(n, d, seed=n + k + per)
    rs = np.append(np.arange(0, n, per), n).astype(np.int32)
    rs[5] = rs[4]                                        # an empty one
    oi, od = oracle.knn(x, rs, k)
    gi, gd = run(x, rs, k, algo=0)
    assert np.array_equal(gi, oi) and np.array_equal(gd, od.view(np.uint32))
