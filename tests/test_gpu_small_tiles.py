"""Launches that take binning tiles of 1024 or 2048 records (the default
binning width, few records): a record short of, at and past each tile and each
change of width, fused with their answers and as a separate insert, against
the oracle; and the same records at an explicit width."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu
RTOL = 1e-5


def _records(n, seed):
    rng = np.random.default_rng(seed)
    p = rng.uniform(-2.0, 2.0, (3, n))
    run = np.arange(n) // 5 * 5  # five neighbouring records share a vertex: runs across wave and tile ends
    nrm = rng.normal(size=(3, n))
    v = rng.exponential(size=(3, n))
    v[1, rng.random(n) < 0.01] = np.nan
    return records(n, px=p[0, run], py=p[1, run], pz=p[2, run], nx=nrm[0, run], ny=nrm[1, run], nz=nrm[2, run],
                   r=v[0], g=v[1], b=v[2])


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2049, 8192, 512 * 1024, 512 * 1024 + 1, 1024 * 1024 + 3])
def test_small_launches_match_the_oracle(n):
    import oracle
    from paper_2005_07547_amd import psf
    cfg = dict(log2_slots=16, e_min=-2, kappa=0.0, normal_bins_log2=0)  # 4096 cells
    tabs = [psf.Table(**cfg, max_batch=n), psf.Table(**cfg, max_batch=n, bin_per=8), psf.Table(**cfg)]
    orc = oracle.Oracle(**cfg)
    for it in range(2):
        rec = _records(n, 10 * it + 1)
        d = to_device(rec)
        out, found = tabs[0].iterate(d)
        out8, found8 = tabs[1].iterate(d)
        tabs[2].insert(d)
        tabs[2].update()
        orc.insert(rec)
        orc.update()
        want, hit = orc.query(rec)
        for o, f in ((out, found), (out8, found8), tabs[2].query(d)):
            assert np.array_equal(f.cpu().numpy(), hit)
            err = np.abs(o.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-30)
            assert float(err[:, hit.astype(bool)].max(initial=0.0)) <= RTOL
    cells = orc.export()
    for t in tabs:
        ex = t.export()
        assert np.array_equal(ex["keys"], cells["keys"])
        assert np.array_equal(ex["c_old"].astype(np.uint64), cells["c_old"])
        assert t.stats()["dropped"] == 0
