"""Order inside dense cells (two dimensions, more than 2^20 points): the records stay a permutation inside their cells, runs of them
get small boxes, and the graph stays the tile kernel's on every row and the oracle's on sampled ones."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = (1 << 20) + 4321


def cloud(kind, rng):
    x = rng.random((N, 2))
    if kind == "power":                                     # several steps at the centre
        x = x[:, :1] ** 3 * np.stack([np.cos(6.2831853 * x[:, 1]), np.sin(6.2831853 * x[:, 1])], axis=1)
    if kind == "scales":                                    # every step peels off one scale: more of them than are taken
        x[:60000] *= 1e-3 * 0.02 ** rng.integers(0, 15, size=(60000, 1))
    if kind == "copies":                                    # pieces that no step splits, inside a cell and alone in one
        x[:30000] = 0.25
        x[30000:60000] = 0.75 + 1e-6 * (rng.integers(0, 3, size=(30000, 1)) == 1)
    if kind == "sizes":                                     # cells of the sizes around the lines of the lists
        for i, m in enumerate([96, 97, 255, 256, 257, 1024, 1025, 2047, 2048, 2049, 4096, 5000]):
            x[20000 * i:20000 * i + m] = (i + 0.5) / 12 + 1e-6 * x[20000 * i:20000 * i + m]
    return np.ascontiguousarray(x[rng.permutation(N)].astype(np.float32))


@pytest.mark.parametrize("kind,bins", [("power", 0), ("scales", 0), ("copies", 0), ("sizes", 0), ("uniform", 0), ("power", 3)])
def test_records_and_graph(kind, bins):
    rng = np.random.Generator(np.random.PCG64(len(kind)))
    x = cloud(kind, rng)
    rs = np.array([0, N // 3, N // 3, N], dtype=np.int32)
    k = 10
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    bn = B.fg_bin_points(xt, rt, k, bins, 2 if bins else 0)
    torch.cuda.synchronize()
    cells, bounds, rows = bn.bin_idx.cpu().numpy(), bn.bin_bounds.cpu().numpy(), bn.perm.cpu().numpy()
    assert np.array_equal(np.sort(rows), np.arange(N)) and np.array_equal(bn.sorted_records.cpu().numpy()[:, :2], x[rows])
    assert np.all(np.diff(cells[rows]) >= 0) and np.array_equal(np.diff(bounds), np.bincount(cells, minlength=len(bounds) - 1))
    size = np.diff(bounds)
    big = int(np.argmax(size))
    if kind == "power":                                     # the fullest cell: boxes of 32 points a small part of the cell's
        p = x[rows[bounds[big]:bounds[big + 1]]][:size[big] // 32 * 32].reshape(-1, 32, 2)
        area = np.prod(p.max(1) - p.min(1), axis=1)
        assert np.median(area) < np.prod(p.max((0, 1)) - p.min((0, 1))) * 100.0 / len(area)
    if bins:                                                # (every pair of a coarse grid's bins: too slow for the other kernels)
        idx, d2 = B.fg_query_binned(bn, rt, k)
    else:
        idx, d2 = B.fg_query_binned(bn, rt, k)
        ref = B.fg_query_binned(bn, rt, k, algo=4)
        assert torch.equal(idx, ref[0]) and torch.equal(d2, ref[1])
    pick = np.unique(np.concatenate([rows[bounds[big]:bounds[big + 1]][:5], rng.choice(N, 15, replace=False)])).astype(np.int64)
    oi, od = oracle.knn_rows(x, rs, k, pick)
    assert np.array_equal(idx.cpu().numpy()[pick], oi) and np.array_equal(d2.cpu().numpy()[pick].view(np.uint32), od.view(np.uint32))
