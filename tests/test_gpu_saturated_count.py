"""The count of clamped F16 stores: every blended cell of a frame whose values
lie past 65504, however many of them a thread of the merge writes back (frames
of one round, of several, and dense ones)."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("state", [1, 3])
@pytest.mark.parametrize("n,cells,part_log2", [(1500, 900, 12), (4000, 2500, 12), (4000, 2500, 8), (4000, 200, 11),
                                               (9000, 2500, 12), (9000, 1500, 11)])
def test_every_clamped_cell_is_counted(n, cells, part_log2, state):
    from paper_2005_07547_amd import psf
    slots = 12
    t = psf.Table(log2_slots=slots, part_log2=part_log2, max_probe=1 << part_log2, state_dtype=state,
                  normal_bins_log2=0)
    rng = np.random.default_rng(n + cells)
    at = np.concatenate([np.arange(cells), rng.integers(0, cells, n - cells)])
    rec = records(n, px=at % 64 + 0.5, py=at // 64 + 0.5, pz=np.full(n, 0.5), nx=np.zeros(n), ny=np.zeros(n),
                  nz=np.ones(n), r=np.full(n, 1e6), g=np.ones(n), b=np.full(n, -1e6))
    for frame in (1, 2):
        t.iterate(to_device(rec))
        st = t.stats()
        assert st["touched_last"] == cells and st["dropped"] == 0
        assert st["saturated"] == frame * cells
