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
