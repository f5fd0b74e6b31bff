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
