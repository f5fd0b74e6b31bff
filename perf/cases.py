"""Workloads of the Friends-of-Friends labelling, as user programs call it.

A case is one way of calling the library (``how``) on one kind of particle
distribution (``what``): the one-shot call, a kept handle fed new snapshots,
a captured graph, a batch of boxes, the entry point that allocates nothing,
new linking lengths over built cells, and the group catalogue. Sizes run from
the thousand particles of the smallest box of the batch workload to the 3.4e7
of the whole batch. Inputs are made on the GPU: Plummer halos with counts from
M^-1.9 over a uniform background (60 % of the particles in halos unless the
case says otherwise), uniform points, or the sites of a lattice with
vacancies, nearly all of which form one group.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2003_11468_amd as fof

# the autotuner's choice for the clustered workloads (cells of 1.375 l_x,
# cells of 16 particles searched by whole wavefronts, 4096 work-groups there)
TUNED = {"cell_factor": 1.375, "dense_min": 16, "schedule": 8}


def _case(name=None, how="run", what="clustered", n=100_000, n_boxes=1, n_min=0, b=0.2, halos=0.6, box=1.0,
          predicate="fp32_filter", strict=False, tuned=False, domains=0, ratio=1.0, min_size=20):
    """One case; `n` is the size of a box, or the upper end of a batch's log-uniform sizes from n_min."""
    c = {"how": how, "what": what, "n": int(n), "n_boxes": int(n_boxes), "n_min": int(n_min), "b": float(b),
         "halos": float(halos), "box": float(box), "predicate": predicate, "strict": bool(strict),
         "tuned": bool(tuned), "domains": int(domains), "ratio": float(ratio), "min_size": int(min_size)}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a first look at a small cutout: the one-shot call, handle and workspace made inside it
        _case("label_1k", "label", "clustered", 1000),
        # the smoke workload, a handle fed one uniform snapshot after another
        _case("run_uniform_32k", "run", "uniform", 32 ** 3),
        # a zoom region labelled inside a loop that may not allocate; odd size
        _case("noalloc_100k", "noalloc", "clustered", 100_003),
        # a batch of small boxes (cutouts around candidates), eager
        _case("boxes_64_small", "run", "clustered", 30_000, n_boxes=64, n_min=1000),
        # the plain double predicate with `<`, a box in Mpc, odd size
        _case("run_fp64_1m", "run", "clustered", 1_000_003, box=25.0, predicate="fp64", strict=True),
        # one snapshot with the default options
        _case("run_clustered_2m", "run", "clustered", 128 ** 3),
        # nearly every particle in one group: the contention the union-find has to survive
        _case("run_lattice_2m", "run", "lattice", 128 ** 3),
        # the on-the-fly finder: a second linking length over the cells of the last run
        _case("relink_2m", "relink", "clustered", 128 ** 3, tuned=True, ratio=0.8),
        # groups above 20 members of labels in hand
        _case("catalogue_4m", "catalogue", "clustered", 4_000_037),
        # a large snapshot with the default options
        _case("run_clustered_16m", "run", "clustered", 256 ** 3),
        # the same in a graph with the tuned options, a simulation's fixed buffers
        _case("graph_clustered_16m", "graph", "clustered", 256 ** 3, tuned=True),
        # the headline: 256 boxes of 1e3 to 1e6 particles in one graph
        _case("graph_batch_256", "graph", "clustered", 1_000_000, n_boxes=256, n_min=1000, tuned=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    how = rng.choice(["label", "run", "run", "run", "noalloc", "graph", "batch", "relink", "catalogue"])
    what = rng.choice(["clustered", "clustered", "clustered", "uniform", "lattice"])
    tuned = rng.random() < 0.5
    top = {"label": 1_000_000, "noalloc": 1_000_000, "relink": 8_000_000, "catalogue": 8_000_000}.get(
        how, 16_000_000 if tuned else 6_000_000)
    n = _log_int(rng, 1000, top)
    kw = {"b": round(rng.uniform(0.15, 0.3), 3), "halos": rng.choice([0.6, 0.7, 0.9]), "box": rng.choice([1.0, 25.0, 100.0]),
          "predicate": rng.choice(["fp32_filter", "fp32_filter", "fp64"]), "strict": rng.random() < 0.2}
    if how == "batch":
        # with the default options whole batches of large boxes cost more than the headline
        return _case(how=rng.choice(["run", "graph"]), what="clustered", n=_log_int(rng, 2000, 500_000 if tuned else 60_000),
                     n_boxes=_log_int(rng, 2, 256), n_min=1000, tuned=tuned, **kw)
    if how in ("label", "noalloc"):
        return _case(how=how, what=what, n=n, **kw)
    if how == "relink":
        return _case(how=how, what="clustered" if what == "lattice" else what, n=n, tuned=tuned,
                     ratio=round(rng.uniform(0.5, 1.0), 3), **kw)
    if how == "catalogue":
        return _case(how=how, what="clustered", n=n, min_size=rng.choice([1, 2, 20, 32, 100]), **kw)
    domains = rng.choice([0, 0, 0, 8]) if how == "run" else 0
    return _case(how=how, what=what, n=n, tuned=tuned, domains=domains, **kw)


# ---------------------------------------------------------------- inputs --

def _halo_counts(r, budget, m_max=1e5, m_min=20.0, slope=1.9):
    """Halo masses from dN/dM ~ M^-slope on [m_min, m_max], the last one clipped to the budget."""
    out, left = [], int(budget)
    a, lo, hi = 1.0 - slope, m_min ** (1.0 - slope), m_max ** (1.0 - slope)
    while left > 0:
        m = np.rint((lo + (hi - lo) * r.random(4096)) ** (1.0 / a)).astype(np.int64)
        c = np.cumsum(m)
        k = int(np.searchsorted(c, left))
        out.append(m[:k + 1])
        if k < len(m):
            out[-1][-1] -= int(c[k]) - left
            left = 0
        else:
            left -= int(c[-1])
    m = np.concatenate(out) if out else np.zeros(0, np.int64)
    return m[m > 0]


def _clustered(sizes, halos, r, g, dev):
    """Unit-box positions (float64) of every box, each box's particles in shuffled order."""
    per_box = [_halo_counts(r, round(halos * s)) for s in sizes]
    counts = np.concatenate(per_box)
    halo_box = np.repeat(np.arange(len(sizes)), [len(c) for c in per_box])
    background = sizes - np.bincount(halo_box, weights=counts, minlength=len(sizes)).astype(np.int64)
    m = torch.from_numpy(counts).to(dev)
    centre = torch.rand(len(counts), 3, dtype=torch.float64, device=dev, generator=g)
    scale = 0.005 * (m.double() / 1000.0) ** (1.0 / 3.0)
    of = torch.repeat_interleave(torch.arange(len(counts), device=dev), m)
    u = 0.999 * (1.0 - torch.rand(len(of), dtype=torch.float64, device=dev, generator=g))
    rad = scale[of] * (u ** (-2.0 / 3.0) - 1.0) ** -0.5
    cos = 2.0 * torch.rand(len(of), dtype=torch.float64, device=dev, generator=g) - 1.0
    phi = 2.0 * math.pi * torch.rand(len(of), dtype=torch.float64, device=dev, generator=g)
    sin = torch.sqrt(1.0 - cos * cos)
    unit = torch.stack([sin * torch.cos(phi), sin * torch.sin(phi), cos], dim=1)
    inside = centre[of] + rad[:, None] * unit
    inside = inside - torch.floor(inside)
    outside = torch.rand(int(background.sum()), 3, dtype=torch.float64, device=dev, generator=g)
    box_in = torch.from_numpy(halo_box).to(dev)[of]
    box_out = torch.repeat_interleave(torch.arange(len(sizes), device=dev), torch.from_numpy(background).to(dev))
    pos, box = torch.cat([inside, outside]), torch.cat([box_in, box_out])
    order = torch.argsort(box.double() + torch.rand(len(pos), dtype=torch.float64, device=dev, generator=g))
    return pos[order]


def _positions(case, sizes, seed, dev):
    """FP32 positions in [0, L) and the linking length of every box."""
    r = np.random.RandomState(seed % (1 << 32))
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    n = int(sizes.sum())
    L = case["box"]
    lx = case["b"] * L / np.cbrt(sizes.astype(np.float64))
    if case["what"] == "uniform":
        pos = torch.rand(n, 3, dtype=torch.float64, device=dev, generator=g)
    elif case["what"] == "lattice":
        # 60 % of the sites of a lattice, 0.9 l_x apart and moved by up to 2 % of that: the six
        # axis neighbours link, and with so many sites taken one group spans the box
        side = math.ceil((n / 0.6) ** (1.0 / 3.0))
        s = torch.randperm(side ** 3, device=dev, generator=g)[:n]
        site = torch.stack([s % side, (s // side) % side, s // (side * side)], dim=1).double()
        move = 0.04 * (torch.rand(n, 3, dtype=torch.float64, device=dev, generator=g) - 0.5)
        pos = (site + 0.5 + move) / side
        lx = np.array([L / side / 0.9])
    else:
        pos = _clustered(sizes, case["halos"], r, g, dev)
    pos = (pos * L).float()
    pos[pos >= L] = 0.0   # a coordinate rounded up to L is its periodic image
    return pos.contiguous(), lx


def _sizes(case):
    if case["n_boxes"] > 1:
        # the batch's sizes stay the same from snapshot to snapshot, as the graph of a batch does
        r = np.random.RandomState(3)
        u = r.uniform(math.log(case["n_min"]), math.log(case["n"]), case["n_boxes"])
        return np.rint(np.exp(u)).astype(np.int64)
    return np.array([case["n"]], dtype=np.int64)


def prepare(case, seed):
    dev = torch.device("cuda")
    sizes = _sizes(case)
    offsets = np.zeros(len(sizes) + 1, dtype=np.int64)
    offsets[1:] = np.cumsum(sizes)
    pos, lx = _positions(case, sizes, seed, dev)
    n = len(pos)
    box = np.full(len(sizes), case["box"])
    s = {"case": case, "how": case["how"], "pos": pos, "offsets": offsets, "box": box, "lx": lx,
         "label": torch.empty(n, dtype=torch.int32, device=dev), "size": torch.empty(n, dtype=torch.int32, device=dev)}
    opt = dict(TUNED) if case["tuned"] else {}
    opt.update(predicate=case["predicate"], strict=case["strict"])
    if case["how"] == "label":
        return s
    if case["how"] == "noalloc":
        s["opt"] = fof.make_options(**opt)
        s["stream"] = torch.cuda.current_stream().cuda_stream
        return s
    f = s["f"] = fof.FoF(domains=case["domains"], **opt)
    f.reserve(offsets, box, lx)
    if case["how"] == "graph":
        f.capture(pos, offsets, box, lx, s["label"], s["size"])
    elif case["how"] in ("relink", "catalogue"):
        f.run(pos, offsets, box, lx, s["label"], s["size"])
        s["lx2"] = lx * case["ratio"]
        if case["how"] == "catalogue":   # arrays as long as the groups of that size can be many
            s["cat"] = [torch.zeros(n // case["min_size"] + 1, dtype=torch.int32, device=dev) for _ in range(3)]
    return s


def run(s):
    c, how = s["case"], s["how"]
    if how == "label":
        label, size, n_groups = fof.label(s["pos"], float(s["lx"][0]), box=c["box"], predicate=c["predicate"],
                                          strict=c["strict"])
        return {"label": label, "size": size, "n_groups": n_groups}
    if how == "noalloc":   # ordered on the stream, nothing read back
        fof.fof_label_noalloc(s["pos"], c["box"], float(s["lx"][0]), s["label"], s["size"], s["opt"], s["stream"],
                              sync=False)
        return {"label": s["label"], "size": s["size"]}
    f = s["f"]
    if how == "graph":
        f.replay()
        return {"label": s["label"], "size": s["size"]}
    if how == "relink":
        label, size, n_groups = f.relink(s["lx2"], len(s["lx"]), s["label"], s["size"])
        return {"label": label, "size": size, "n_groups": n_groups}
    if how == "catalogue":
        first, size, box = s["cat"]
        count = fof.fof_catalogue(f.ctx, s["label"], s["size"], c["min_size"], first, size, box, len(first))
        return {"first": first, "size": size, "box": box, "count": count}
    label, size, n_groups = f.run(s["pos"], s["offsets"], s["box"], s["lx"], s["label"], s["size"])
    return {"label": label, "size": size, "n_groups": n_groups}


def work(case):
    """Positions read once, labels and sizes written once; a relink reads and
    writes the same, a catalogue reads the sizes."""
    n = int(_sizes(case).sum())
    return {"bytes": (4 if case["how"] == "catalogue" else 20) * n, "flops": 0}


def exact(case, seed):
    return None   # labels, sizes and counts are whole numbers: they are equal or wrong
