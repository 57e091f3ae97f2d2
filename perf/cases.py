"""Cases of use of the exact k-nearest-neighbour graph build, with their inputs and the work they cannot do without.

Each case is one pass through the public calls of ``paper_2511_10442_amd.binding`` as a program that builds graphs
makes them: inputs on the GPU, workspace and output tensors kept from one pass to the next.

``op``
    forward   fg_binned_select_knn: the graph alone (inference, graph construction for a fixed cloud)
    dir       fg_binned_select_knn_dir: some points only ask, some only answer
    step      a training step that bins its points once: fg_bin_points, fg_query_binned, fg_knn_backward_binned
    autograd  a training step whose two halves know nothing of each other: fg_binned_select_knn, fg_knn_backward
    oc        fg_oc_helper: the index matrices of the object-condensation loss
``cloud``
    uniform   independent uniform coordinates: the published benchmark's input
    mixture   50 Gaussian clusters over a uniform background: a learned latent space
    showers   anisotropic clusters of ~450 points over noise: detector hits
    skewed    density that falls with a power of the radius, plus 1000 narrow hotspots
"""
import math

import numpy as np
import torch

from paper_2511_10442_amd import binding as fg

_MAX_SLOTS = 200_000_000      # n * k of the largest forward case
_MAX_STEP_SLOTS = 80_000_000  # n * k of the largest training step
_MAX_OC_WORDS = 200_000_000   # entries of the largest M_not


def listed():
    return [
        # one small event in an online reconstruction: latency and launches are all there is
        _knn("event_1k_d3_k10", "forward", "uniform", 1000, 3, 10),
        # a batch of small ragged events, latent space of four dimensions, the two halves of the step apart
        _knn("ragged_20k_d4_k24_autograd", "autograd", "mixture", 20011, 4, 24, splits=48, ragged=True),
        # two clustered events in a learned space, training step
        _knn("mixture_100k_d4_k40_step", "step", "mixture", 100000, 4, 40, splits=2),
        # a batch of ten detector events of 100k hits, training step: the headline workload
        _knn("showers_1m_d3_k32_step", "step", "showers", 1000000, 3, 32, splits=10),
        # strongly varying density, many short rows, training step
        _knn("skewed_5m_d2_k16_step", "step", "skewed", 5000000, 2, 16, splits=5),
        # the published sweep over sizes, its large end
        _knn("uniform_5m_d3_k40", "forward", "uniform", 5000000, 3, 40),
        # the published sweep over k, its largest k: more neighbours than one sorted list holds
        _knn("uniform_100k_d3_k100", "forward", "uniform", 100000, 3, 100),
        # the published sweep over dimensions: in the middle, and at its far end
        _knn("uniform_1m_d5_k40", "forward", "uniform", 1000000, 5, 40),
        _knn("uniform_500k_d8_k64", "forward", "uniform", 500000, 8, 64),
        _knn("uniform_60k_d10_k40", "forward", "uniform", 60001, 10, 40),
        # hits of three events of which some only look for neighbours and some are only found
        _knn("showers_300k_d3_k20_dir", "dir", "showers", 300007, 3, 20, splits=3, ragged=True),
        # the loss's index matrices for a batch of ten events with 200 objects each
        _oc("oc_10x100k_200", 10, 100000, 200),
    ]


def draw(rng):
    if rng.random() < 0.1:
        splits = rng.randint(1, 10)
        size = _log_int(rng, 1000, 100000)
        objects = _log_int(rng, 10, 200)
        while splits * objects * size > _MAX_OC_WORDS:
            objects = max(1, objects // 2)
        return _oc(None, splits, size, objects)
    cloud = rng.choice(["uniform", "uniform", "uniform", "mixture", "mixture", "showers", "showers", "skewed"])
    op = rng.choice(["forward", "forward", "step", "step", "autograd", "dir"])
    d = {"uniform": rng.randint(2, 10), "mixture": rng.randint(3, 6), "showers": 3, "skewed": 2}[cloud]
    # sizes stay where the cost per query, which grows quickly with the dimension, leaves a pass below the largest listed one
    most = {2: 5_000_000, 3: 5_000_000, 4: 2_000_000, 5: 1_000_000, 6: 400_000, 7: 400_000, 8: 400_000, 9: 60_000, 10: 50_000}[d]
    if cloud == "mixture":
        most = min(most, 200_000)
    k = _log_int(rng, 8, 100 if d <= 4 else (64 if d <= 8 else 40))
    if cloud == "skewed":
        k = min(k, 32)
        most = 3_000_000
    slots = _MAX_STEP_SLOTS if op in ("step", "autograd") else _MAX_SLOTS
    n = min(_log_int(rng, 1000, most), slots // k)
    splits = min(_log_int(rng, 1, 64), max(1, n // 200))
    return _knn(None, op, cloud, n, d, k, splits=splits, ragged=rng.random() < 0.5)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _knn(name, op, cloud, n, d, k, splits=1, ragged=False):
    case = {"op": op, "cloud": cloud, "n": n, "d": d, "k": k, "splits": splits, "ragged": ragged}
    return dict(case, name=name) if name else case


def _oc(name, splits, size, objects):
    case = {"op": "oc", "splits": splits, "size": size, "objects": objects}
    return dict(case, name=name) if name else case


def work(case):
    if case["op"] == "oc":
        # every association read once, both matrices written once (an object's row of M holds its ~size/objects members)
        n, u = case["splits"] * case["size"], case["splits"] * case["objects"]
        return {"bytes": 4.0 * (n + u * case["size"] + n), "flops": 0.0}
    n, d, k = case["n"], case["d"], case["k"]
    nbytes = 4.0 * n * d + 8.0 * n * k          # coordinates in; indices and squared distances out
    flops = n * k * (3.0 * d - 1)               # the distances that are returned
    if case["op"] == "dir":
        nbytes += 4.0 * n
    if case["op"] in ("step", "autograd"):
        nbytes += 4.0 * n * k + 4.0 * n * d     # upstream gradient in, coordinate gradient out
        flops += n * k * 4.0 * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Graphs, distances and index matrices are defined to the bit.  Gradients are sums of some 2 k float32 terms,
    # each sum rounded to float32 a few times: against sums in double precision they are off by 8e-8 (2-norm) and at
    # most 1.1e-6 of the larger of the value and the result's root mean square; four to five times that.
    if case["op"] in ("step", "autograd"):
        return {"rel": 4e-7, "max": 5e-6}
    return "exact"


# ---- inputs ------------------------------------------------------------------------------------------------

def _sizes(case, rng):
    n, s = case["n"], case["splits"]
    if not case["ragged"]:
        return [n // s + (1 if i < n % s else 0) for i in range(s)]
    cuts = np.sort(rng.integers(0, n + 1, size=s - 1))
    return np.diff(np.concatenate([[0], cuts, [n]])).astype(int).tolist()


def _cloud(case, sizes, rng, gen):
    n, d, dev = case["n"], case["d"], "cuda"

    def rand(*shape):
        return torch.rand(*shape, generator=gen, device=dev, dtype=torch.float64)

    def randn(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float64)

    if case["cloud"] == "uniform":
        return rand(n, d).float()
    if case["cloud"] == "mixture":
        x = rand(50, d)[torch.randint(0, 50, (n,), generator=gen, device=dev)] * 10.0 + 0.3 * randn(n, d)
        noise = rand(n, 1) < 0.1
        return torch.where(noise, rand(n, d) * 10.0, x).float()
    if case["cloud"] == "skewed":
        r, a = rand(n) ** 3, rand(n) * (2.0 * math.pi)
        x = torch.stack([r * torch.cos(a), r * torch.sin(a)], dim=1)
        split = torch.repeat_interleave(torch.arange(len(sizes), device=dev), torch.tensor(sizes, device=dev))
        spot = split * 1000 + torch.randint(0, 1000, (n,), generator=gen, device=dev)
        hot = (rand(len(sizes) * 1000, 2) * 2.0 - 1.0)[spot] + 1e-3 * randn(n, 2)
        return torch.where(rand(n, 1) < 0.4, hot, x).float()
    # showers: one per ~500 points of a split; nine points in ten belong to one
    counts = [max(1, s // 500) for s in sizes]
    first = np.concatenate([[0], np.cumsum(counts)])
    total = int(first[-1])
    basis, _ = np.linalg.qr(rng.standard_normal((total, 3, 3)))
    sigma = np.exp(rng.uniform(math.log(0.01), math.log(0.5), size=(total, 3)))
    shape = torch.from_numpy(basis * sigma[:, None, :]).to(dev)      # columns scaled by the axis widths
    split = torch.repeat_interleave(torch.arange(len(sizes), device=dev), torch.tensor(sizes, device=dev))
    lo = torch.from_numpy(first[:-1].copy()).to(dev)[split]
    number = torch.from_numpy(np.asarray(counts)).to(dev)[split]
    which = lo + (rand(n) * number).long().clamp_(max=max(counts) - 1).minimum(number - 1)
    centre = rand(total, 3) * 10.0
    x = centre[which] + torch.einsum("nij,nj->ni", shape[which], randn(n, 3))
    noise = rand(n, 1) < 0.1
    return torch.where(noise, rand(n, 3) * 10.0, x).float()


def _prepare_oc(case, gen):
    dev = "cuda"
    splits, size, objects = case["splits"], case["size"], min(case["objects"], case["size"])
    n = splits * size
    asso = torch.empty(n, dtype=torch.int64, device=dev)
    unique = []
    for s in range(splits):
        points = torch.randperm(size, generator=gen, device=dev)[:objects].sort().values + s * size
        weight = torch.rand(objects, generator=gen, device=dev) ** 3 + 1e-3
        edge = torch.cumsum(weight, 0) / weight.sum()
        pick = torch.searchsorted(edge, torch.rand(size, generator=gen, device=dev)).clamp_(max=objects - 1)
        a = points[pick]
        a[torch.rand(size, generator=gen, device=dev) < 0.1] = -1
        a[points - s * size] = points             # a condensation point belongs to itself
        asso[s * size:(s + 1) * size] = a
        unique.append(points)
    members = min(size, 5 * size // objects + 32)   # room for the largest object: weights reach four times their mean
    u = splits * objects
    return {"op": "oc", "asso": asso.int(), "unique": torch.cat(unique).int(),
            "unique_rs": torch.repeat_interleave(torch.arange(splits, device=dev), objects).int(),
            "rs": torch.arange(splits + 1, device=dev, dtype=torch.int32) * size, "maxuq": members, "maxrs": size,
            "M": torch.empty((members, u), dtype=torch.int32, device=dev),
            "M_not": torch.empty((size, u), dtype=torch.int32, device=dev),
            "ws": torch.empty(max(256, fg.fg_oc_helper_workspace_size(u, size)), dtype=torch.uint8, device=dev)}


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if case["op"] == "oc":
        return _prepare_oc(case, gen)
    rng = np.random.default_rng(int(seed))
    n, d, k = case["n"], case["d"], case["k"]
    sizes = _sizes(case, rng)
    state = {"op": case["op"], "k": k, "x": _cloud(case, sizes, rng, gen).contiguous(),
             "rs": torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).cuda(),
             "ws": fg.alloc_workspace(n, d, len(sizes), k),
             "idx": torch.empty((n, k), dtype=torch.int32, device="cuda"),
             "d2": torch.empty((n, k), dtype=torch.float32, device="cuda")}
    if case["op"] == "dir":
        # three points in five both ask and answer, one in five only asks, one in five only answers
        roll = torch.rand(n, generator=gen, device="cuda")
        state["dir"] = torch.where(roll < 0.6, 3, torch.where(roll < 0.8, 1, 0)).int()
    if case["op"] in ("step", "autograd"):
        state["g"] = torch.randn((n, k), generator=gen, device="cuda")
        state["grad"] = torch.empty((n, d), dtype=torch.float32, device="cuda")
    return state


def run(state):
    op = state["op"]
    if op == "oc":
        return fg.fg_oc_helper(state["asso"], state["unique"], state["unique_rs"], state["rs"], state["maxuq"],
                               state["maxrs"], M=state["M"], M_not=state["M_not"], workspace=state["ws"])
    x, rs, k, ws, idx, d2 = (state[name] for name in ("x", "rs", "k", "ws", "idx", "d2"))
    if op == "dir":
        return fg.fg_binned_select_knn_dir(x, rs, state["dir"], k, workspace=ws, out_idx=idx, out_d2=d2)
    if op == "step":
        binning = fg.fg_bin_points(x, rs, k, workspace=ws)
        fg.fg_query_binned(binning, rs, k, idx, d2)
        return idx, d2, fg.fg_knn_backward_binned(binning, state["g"], idx, x, state["grad"])
    fg.fg_binned_select_knn(x, rs, k, workspace=ws, out_idx=idx, out_d2=d2)
    if op == "autograd":
        return idx, d2, fg.fg_knn_backward(state["g"], idx, x, rs, state["grad"], ws)
    return idx, d2
