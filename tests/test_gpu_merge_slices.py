"""Launches of fewer, as many and a few more tiles than a merge block has
wavefronts, with the run table read in place and transposed, against the
oracle."""
import numpy as np
import pytest

from tests.helpers import to_device
from tests.test_gpu_small_tiles import RTOL, _records

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("tiles", [1, 3, 11, 12, 13, 25])
def test_few_tiles_match_the_oracle(tiles, transposed):
    import oracle
    from paper_2005_07547_amd import psf
    cfg = dict(log2_slots=16, e_min=-2, kappa=0.0, normal_bins_log2=0)
    n = (tiles - 1) * 4096 + 1  # one record in the last tile
    tab = psf.Table(**cfg, max_batch=n, bin_per=8, part_log2=12,
                    flags=psf.PSF_FLAG_TRANSPOSE_RUNS if transposed else 0)
    orc = oracle.Oracle(**cfg)
    for it in range(2):
        rec = _records(n, 7 * it + tiles)
        out, found = tab.iterate(to_device(rec))
        orc.insert(rec)
        orc.update()
        want, hit = orc.query(rec)
        assert np.array_equal(found.cpu().numpy(), hit)
        err = np.abs(out.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-30)
        assert float(err[:, hit.astype(bool)].max(initial=0.0)) <= RTOL
    ex, cells = tab.export(), orc.export()
    assert np.array_equal(ex["keys"], cells["keys"])
    assert np.array_equal(ex["c_old"].astype(np.uint64), cells["c_old"])
