"""The binning of few points (one launch, 16-bit counters in LDS) and the general one, on both sides of the line between them,
against the definition in numpy float32: cells, boundaries, geometry and records, and the backward's own row order."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B
from paper_2511_10442_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def expected_cells(x, rs, n_bins, d_bin, sub):
    cells = np.zeros(len(x), dtype=np.int64)
    per_split = n_bins ** d_bin * sub
    for s in range(len(rs) - 1):
        p = x[rs[s]:rs[s + 1], :d_bin]
        if len(p) == 0:
            continue
        flat = np.zeros(len(p), dtype=np.int64)
        for c in range(d_bin):
            nb = n_bins * sub if c == d_bin - 1 else n_bins
            lo, hi = p[:, c].min(), p[:, c].max()
            ext = np.float32(hi - lo)
            inv = np.float32(nb) / ext if ext >= np.float32(1e-30) else np.float32(0)
            j = np.floor((p[:, c] - lo) * inv).astype(np.int64)
            flat = flat * nb + np.clip(j, 0, nb - 1)
        cells[rs[s]:rs[s + 1]] = s * per_split + flat
    return cells, per_split


# (sizes, d, n_bins, d_bin): one launch up to 1024 splits, 48,000 cells a split, 49,152 points, and n (d + 8) <= 327,680 a split
@pytest.mark.parametrize("sizes,d,nb,db", [
    ([1], 2, 3, 2), ([0, 2, 0], 3, 5, 3), ([63, 0, 64, 1025], 4, 0, 0), ([5000], 5, 0, 0), ([3000, 17], 3, 7, 3),     # 343 cells and slices
    ([20000], 3, 0, 0), ([29789], 3, 0, 0), ([29790], 3, 0, 0),                     # the line of one split
    ([1] * 1024, 2, 2, 2), ([1] * 1025, 2, 2, 2),                                   # of the splits
    ([14000], 2, 86, 2), ([14000], 2, 87, 2),                                       # of the LDS that is free: 4 x 7396 and 4 x 7569 cells
    ([24000], 2, 109, 2), ([24000], 2, 110, 2), ([25000], 3, 20, 3),                # of the cells: 4 x 11,881 and 4 x 12,100; 4 x 8000
    ([100, 48000, 900, 152], 2, 0, 0), ([100, 48000, 900, 153], 2, 0, 0),           # of the points, nearly all in one split
    ([18000], 10, 0, 0), ([18300], 10, 0, 0)])
@pytest.mark.parametrize("kind", ["uniform", "same", "flat"])
def test_cells_bounds_and_records(sizes, d, nb, db, kind):
    n = sum(sizes)
    x, rs = W.uniform(n, d, seed=n + d, sizes=sizes)
    x = x - np.float32(0.5)
    if kind == "same": x[:] = x[0]                       # one counter takes all
    if kind == "flat": x[:, 0] = 0.25                    # a dimension without extent
    x = np.ascontiguousarray(x)
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    bn = B.fg_bin_points(xt, rt, 12, nb, db)
    torch.cuda.synchronize()
    cells, per_split = expected_cells(x, rs, bn.n_bins, bn.d_bin, bn.sub_bins)
    got, bounds = bn.bin_idx.cpu().numpy(), bn.bin_bounds.cpu().numpy()
    assert per_split == bn.cells_per_segment and np.array_equal(got, cells)
    assert np.array_equal(np.diff(bounds), np.bincount(cells, minlength=len(bounds) - 1)) and bounds[0] == 0 and bounds[-1] == n
    rec, rows = bn.sorted_records.cpu().numpy(), bn.perm.cpu().numpy()
    assert np.array_equal(np.sort(rows), np.arange(n)) and np.all(np.diff(cells[rows]) >= 0)
    assert np.array_equal(rec[:, :d], x[rows])
    # the backward sorts its rows by a binning of its own
    k = min(4, n)
    rng = np.random.Generator(np.random.PCG64(n))
    idx = rng.integers(0, n, size=(n, k)).astype(np.int32)
    g = rng.standard_normal((n, k)).astype(np.float32)
    grad = B.fg_knn_backward(torch.from_numpy(g).to(DEV), torch.from_numpy(idx).to(DEV), xt, rt, workspace=B.alloc_workspace(n, d, len(rs) - 1, k))
    torch.cuda.synchronize()
    ref, asum = oracle.knn_backward(g, idx, x)
    assert np.all(np.abs(grad.cpu().numpy() - ref) <= 1e-5 * np.maximum(np.abs(ref), asum) + 1e-30)


# the bounding boxes of many points: more points a thread from 393,216 a row split on, chunks that end in the middle of a wavefront and
# straddle a split
@pytest.mark.parametrize("sizes", [[393_216], [393_217], [800_001], [500_000, 0, 7, 1_000_100]])
@pytest.mark.parametrize("d", [2, 5])
def test_boxes_of_many_points(sizes, d):
    n = sum(sizes)
    x, rs = W.uniform(n, d, seed=n, sizes=sizes)
    x[n - 1] = 2.0
    x[rs[-2]] = -1.0                                     # first and last point of the last split hold its box
    bn = B.fg_bin_points(torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV), 12)
    torch.cuda.synchronize()
    cells, _ = expected_cells(x, rs, bn.n_bins, bn.d_bin, bn.sub_bins)
    assert np.array_equal(bn.bin_idx.cpu().numpy(), cells)
