"""GPU parity of the path that compares every pair (up to 4096 points, K <= 65) through each entry point that takes it, and
of the tile kernel at the same sizes, which the default no longer reaches there."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_10442_amd import binding as B
from paper_2511_10442_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# batches of 256 candidates and lanes of 64: sizes around both, the largest size and the first beyond it, the longest list
# and the first that is too long
@pytest.mark.parametrize("sizes", [[1], [2, 0, 63], [64], [65, 255], [256, 257, 1], [1000], [4096], [4097], [1500, 0, 2596]])
@pytest.mark.parametrize("d,k", [(2, 1), (3, 2), (3, 13), (4, 14), (5, 65), (7, 66), (10, 40)])
def test_matches_oracle(sizes, d, k):
    n = sum(sizes)
    x, rs = W.uniform(n, d, seed=n + 7 * d + k, sizes=sizes)
    x[n // 2:n // 2 + 40] = x[n // 2]                # ties
    x = np.ascontiguousarray(x)
    direction = np.random.Generator(np.random.PCG64(n + k)).integers(0, 4, size=n).astype(np.int32)
    xt, rt, dt = (torch.from_numpy(a).to(DEV) for a in (x, rs, direction))
    oi, od = oracle.knn(x, rs, k)
    pi, pd = oracle.knn(x, rs, k, direction=direction)
    bn = B.fg_bin_points(xt, rt, k)
    runs = [(B.fg_binned_select_knn(xt, rt, k), oi, od), (B.fg_binned_select_knn_dir(xt, rt, dt, k), pi, pd),
            (B.fg_query_binned(bn, rt, k), oi, od), (B.fg_query_binned(bn, rt, k, direction=dt), pi, pd),
            (B.fg_query_binned(bn, rt, k, algo=4), oi, od), (B.fg_query_binned(bn, rt, k, direction=dt, algo=4), pi, pd)]
    torch.cuda.synchronize()
    for i, ((gi, gd), ri, rd) in enumerate(runs):
        assert np.array_equal(gi.cpu().numpy(), ri), i
        assert np.array_equal(gd.cpu().numpy().view(np.uint32), rd.view(np.uint32)), i


# what was refused while the small call was binned is still refused
def test_refusals_stay():
    x, rs = W.uniform(500, 3, seed=1)
    xt, rt = torch.from_numpy(x).to(DEV), torch.from_numpy(rs).to(DEV)
    with pytest.raises(Exception):
        B.fg_binned_select_knn(xt, rt, 8, workspace=torch.empty(256, dtype=torch.uint8, device=DEV))
    with pytest.raises(Exception):
        B.fg_binned_select_knn(xt, rt, 8, n_bins=2000, d_bin=3)
    with pytest.raises(Exception):
        B.fg_binned_select_knn(xt, rt, 8, n_bins=4, d_bin=4)
