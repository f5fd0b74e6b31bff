"""Dense cells on the GPU against the CPU oracle, element by element: cells
around the sizes at which their search changes form (64 particles joined in
registers, more by sub-cells; a neighbour of more than 32 that is one group
searched by a sample first), at the box faces and inside, and the automatic
cells that the search subdivides where the workspace holds them.
"""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
fof = pytest.importorskip("paper_2003_11468_amd")

pytestmark = pytest.mark.gpu
LX = 0.09   # eight cells of 1.375 l_x per axis


def blobs(per_cell, spread, seed, corner):
    """per_cell particles in each of 4^3 cells around `corner` (cells wrap at the faces), within `spread` of a
    random point of the cell, and a few in the rest of the box."""
    rng = np.random.default_rng(seed)
    h = 1.0 / 8
    out = [rng.random((200, 3))]
    for c in np.ndindex(4, 4, 4):
        m = int(rng.integers(max(1, per_cell - 1), per_cell + 2))
        centre = rng.random(3)
        local = np.clip(centre + spread * (rng.random((m, 3)) - 0.5), 0.0, 0.999999)
        out.append(((np.array(c) + corner + local) * h) % 1.0)
    pos = np.concatenate(out).astype(np.float32)
    pos[pos >= 1.0] = 0.0
    return pos[rng.permutation(len(pos))]


def run(pos, **kw):
    f = fof.FoF(**kw)
    try:
        label, size, ng = f.run(torch.from_numpy(pos).cuda(), [0, len(pos)], 1.0, LX)
        return label.cpu().numpy(), size.cpu().numpy(), int(ng[0])
    finally:
        f.close()


@pytest.mark.parametrize("predicate", ["fp32_filter", "fp64"])
@pytest.mark.parametrize("spread", [0.15, 1.0])
@pytest.mark.parametrize("per_cell", [8, 16, 17, 32, 33, 64, 65, 150])
def test_cells_around_the_sizes_that_change_the_search(per_cell, spread, predicate):
    for corner in (6, 2):   # across the box faces, and inside
        pos = blobs(per_cell, spread, 7 * per_cell + corner, corner)
        ref = oracle.fof(pos, LX)
        for kw in (dict(dense_min=1), dict(dense_min=8), dict(dense_min=8, schedule=16),
                   dict(dense_min=8, link_order="random"), dict(dense_min=8, compression="depth2"),
                   dict(dense_min=8, domains=3)):
            got = run(pos, predicate=predicate, cell_factor=1.375, **kw)
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and got[2] == ref[2], (corner, kw)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("wrap", [False, True])
def test_one_bridge_between_two_large_groups(axis, wrap):
    """Two cells of one tight group each, too far apart to link but for one
    particle on either side: the sample of a neighbour rarely holds it."""
    rng = np.random.default_rng(5 + axis)
    h = 1.0 / 8
    a, b = np.full(3, 3.5 * h), np.full(3, 3.5 * h)
    face = 0.0 if wrap else 4 * h
    a[axis], b[axis] = face - 0.08, face + 0.08
    pa, pb = (c + 0.004 * (rng.random((300, 3)) - 0.5) for c in (a, b))
    pa[123, axis], pb[211, axis] = face - 0.03, face + 0.03
    for bridge in (True, False):
        pos = np.concatenate([pa, pb if bridge else np.delete(pb, 211, axis=0)]) % 1.0
        pos = pos.astype(np.float32)
        ref = oracle.fof(pos, LX)
        assert ref[2] == (1 if bridge else 2)
        got = run(pos, cell_factor=1.375, dense_min=8)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("predicate", ["fp32_filter", "fp64"])
def test_subdivided_cells_and_a_workspace_that_only_holds_the_coarse_ones(predicate):
    n = 60_000
    pos_np = synth.clustered(n, 9, 0, 0.6)
    lx = synth.linking_length(0.2, n)
    ref = oracle.fof(pos_np, lx)
    pos = torch.from_numpy(pos_np).cuda()
    nc = fof.fof_describe_box(n, 1.0, lx)["cells_per_axis"]
    opt = dict(predicate=predicate)
    coarse = fof.FoF(cell_factor=1.0 / (lx * (nc + 0.5)), dense_min=32, **opt)
    auto = fof.FoF(**opt)
    try:
        assert fof.fof_describe_box(n, 1.0, lx, fof.make_options(cell_factor=1.0 / (lx * (nc + 0.5))))[
            "cells_per_axis"] == nc
        need = fof.fof_workspace_bytes(coarse.ctx, [0, n], 1.0, lx)
        full = fof.fof_workspace_bytes(auto.ctx, [0, n], 1.0, lx)
        assert need < full
        cells = []
        for nbytes in (need, full):
            auto.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
            fof.fof_set_workspace(auto.ctx, auto.ws)
            label, size = auto.outputs(n)
            fof.fof_build_cells(auto.ctx, pos, [0, n], 1.0, lx)
            fof.fof_link(auto.ctx)
            ng = fof.fof_finalize(auto.ctx, label, size, 1)
            assert np.array_equal(label.cpu().numpy(), ref[0]) and np.array_equal(size.cpu().numpy(), ref[1])
            assert int(ng[0]) == ref[2]
            cells.append(auto.stats()["n_cells"])
        assert cells[0] == nc ** 3 < cells[1]
    finally:
        coarse.close()
        auto.close()


def bridged_cells(rng, axis, wrap):
    """Two neighbouring cells of 300 particles, each one set of touching
    sub-cells (a blob, a few particles half way and one near the face), whose
    only link is the pair of particles near the face; and the indices of that pair."""
    h = 1.0 / 8
    face = 0.0 if wrap else 4 * h
    out, at = [], []
    for side in (-1, 1):
        depth = np.full(300, 0.08)
        depth[rng.permutation(300)[:6]] = 0.065   # 0.095 from the other cell's nearest particle
        k = int(rng.integers(300))
        depth[k] = 0.03
        cell = np.full((300, 3), 3.5 * h) + 0.004 * (rng.random((300, 3)) - 0.5)
        cell[:, axis] = face + side * depth + 0.0005 * (rng.random(300) - 0.5)
        at.append(k + 300 * len(out))
        out.append(cell)
    return (np.concatenate(out) % 1.0).astype(np.float32), at


def touching_sets(sub):
    """Number of sets of touching sub-cells (27-neighbourhood) among the rows of `sub`."""
    left, sets = set(map(tuple, sub)), 0
    while left:
        todo, sets = [left.pop()], sets + 1
        while todo:
            c = np.array(todo.pop())
            for d in np.ndindex(3, 3, 3):
                t = tuple(c + np.array(d) - 1)
                if t in left:
                    left.remove(t)
                    todo.append(t)
    return sets


@pytest.mark.parametrize("predicate", ["fp32_filter", "fp64"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("wrap", [False, True])
def test_one_bridge_between_two_cells_of_one_group_each(axis, wrap, predicate):
    """Cells that the pre-merge finds to be one group: a neighbour is sampled
    first, and what the sample misses has to be found in the rest of it."""
    opt = dict(cell_factor=1.375, dense_min=8)
    info = fof.fof_describe_box(600, 1.0, LX, fof.make_options(**opt))
    nc, k = info["cells_per_axis"], info["sub_cells_per_axis"]
    assert nc == 8 and info["sub_cells_adjacent"]
    for seed in range(12):
        rng = np.random.default_rng(100 * seed + 10 * axis + wrap)
        pos, bridge = bridged_cells(rng, axis, wrap)
        cell = np.floor(pos.astype(np.float64) * nc).astype(int)
        sub = np.floor((pos.astype(np.float64) * nc - cell) * k).astype(int)
        cells = np.unique(cell, axis=0)
        assert len(cells) == 2
        for c in cells:
            mine = (cell == c).all(axis=1)
            assert mine.sum() == 300 and touching_sets(sub[mine]) == 1
        for cut in (False, True):
            p = np.delete(pos, bridge[1], axis=0) if cut else pos
            ref = oracle.fof(p, LX)
            assert ref[2] == (2 if cut else 1)
            got = run(p, predicate=predicate, **opt)
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and got[2] == ref[2], (seed, cut)
