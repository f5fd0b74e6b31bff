"""How runs are planned on the host (no device): what planning a batch costs."""
from __future__ import annotations

import time

import numpy as np

import paper_2003_11468_amd as fof


def test_automatic_cells_of_many_boxes_are_counted_in_one_pass():
    """A batch of tiny boxes waits for its planning, so automatic cells, which
    have two sizes to choose from, may not cost two whole plans (7 times the
    plan of given cells; one pass that counts both sizes takes 3 times it,
    most of it their cube roots)."""
    nb = 50_000
    off, side, lx = np.arange(nb + 1, dtype=np.int64) * 20, np.ones(nb), np.full(nb, 0.07)
    cost = {}
    for factor in (0.0, 1.375):
        ctx = fof.fof_create(fof.make_options(cell_factor=factor))
        try:
            took = []
            for _ in range(15):
                t = time.perf_counter()
                fof.fof_workspace_bytes(ctx, off, side, lx)
                took.append(time.perf_counter() - t)
            cost[factor] = min(took)
        finally:
            fof.fof_destroy(ctx)
    assert cost[0.0] < 5.0 * cost[1.375], cost


def test_a_given_segment_size_keeps_its_particles_in_subdivided_cells():
    """segment_log2 counts the cells that the options ask for: where the
    search subdivides them, a run must not be cut into tens of times as many
    segments (each takes a work-group of the sort, and 4 bytes here)."""
    n = 1_000_000
    lx = 0.2 / n ** (1.0 / 3.0)
    cells = fof.fof_describe_box(n, 1.0, lx)["cells_per_axis"] ** 3
    need = {}
    for k in (8, 10, 12, 16):
        ctx = fof.fof_create(fof.make_options(segment_log2=k))
        try:
            need[k] = fof.fof_workspace_bytes(ctx, [0, n], 1.0, lx)
        finally:
            fof.fof_destroy(ctx)
    for k in (8, 10, 12):
        # twice the segments that the cells asked for have, the last segment's
        # occupancy words (8 bytes per 32 cells of at most 2^16) and padding
        assert need[k] - need[16] <= 4 * 2 * (cells >> k) + (1 << 14) + 4096, (k, need)
