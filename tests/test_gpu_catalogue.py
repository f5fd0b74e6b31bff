"""Group catalogues on the GPU around the size at which their launches change,
on given outputs (the catalogue only reads labels and sizes), against torch.
"""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")
fof = pytest.importorskip("paper_2003_11468_amd")

pytestmark = pytest.mark.gpu
LINE = 8192 * 2048   # particles of the most tiles that sum the counts before them themselves


@pytest.mark.parametrize("n", [LINE, LINE + 1, LINE + 2049])
def test_catalogue_on_both_sides_of_the_scan(n):
    gen = torch.Generator(device="cuda").manual_seed(n % 1000)
    pos = torch.rand(n, 3, generator=gen, device="cuda") * 0.999
    size = torch.randint(0, 6, (n,), generator=gen, device="cuda", dtype=torch.int32)
    label = torch.randint(0, n, (n,), generator=gen, device="cuda", dtype=torch.int32)
    size[n - 1] = 5   # the last entry is a group
    offsets = np.array([0, 1_000_001, n], dtype=np.int64)
    f = fof.FoF()
    try:
        f.run(pos, offsets, 1.0, 0.2 / n ** (1.0 / 3.0))   # the catalogue is of the last run's boxes
        for min_size in (1, 5, 6):
            at = torch.nonzero(size >= min_size).flatten()
            first, gsize, box = f.catalogue(label, size, min_size)
            assert torch.equal(first, label[at]) and torch.equal(gsize, size[at])
            assert torch.equal(box, (at >= 1_000_001).to(torch.int32))
        at = torch.nonzero(size >= 3).flatten()
        cap = len(at) - 1   # one entry short: counted, not written
        out = torch.full((2, len(at)), -7, dtype=torch.int32, device="cuda")
        assert fof.fof_catalogue(f.ctx, label, size, 3, out[0], out[1], None, cap) == len(at)
        assert torch.equal(out[0, :cap], label[at[:cap]]) and torch.equal(out[1, :cap], size[at[:cap]])
        assert out[:, cap].tolist() == [-7, -7]
    finally:
        f.close()
