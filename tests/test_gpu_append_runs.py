"""Appends longer than the in-argument cell table: runs of cells in the kernel arguments, or, where the arena is fragmented
into more runs than fit, a table that is uploaded.  Contents are compared bit for bit."""
import numpy as np
import pytest

from gpu_util import Mirror
from paper_2605_26289_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [wl.Shape(8, 2, 128, "bf16"), wl.Shape(4, 1, 64, "bf16"), wl.Shape(6, 3, 64, "f32")])
@pytest.mark.parametrize("counts,accept", [([897], None), ([1, 2000, 0, 3, 700], None), ([1000, 1, 500], [0, 1, 499]),
                                           ([5] * 300, [i % 6 for i in range(300)]), ([4] * 500, None)])
def test_long_appends_land_in_their_cells(shape, counts, accept):
    m = Mirror(shape, len(counts), sum(counts) + 40 * len(counts) + 4096, granule=16, seed=len(counts))
    slots = [m.acquire() for _ in counts]
    m.append(slots, [1 + i % 3 for i in range(len(slots))])  # interleaved growth: runs start inside granules
    m.append(slots, counts, n_accept=accept)
    m.append(slots, [2] * len(slots))
    for s in (slots if len(slots) < 10 else slots[:5] + slots[-5:] + slots[140:145]):
        m.check_gather(s)
    cells = np.concatenate([m.pool.cells(s) for s in slots])
    assert len(set(cells.tolist())) == len(cells)
    m.pool.close()
