"""Batched iterations of few records, whose sessions take binning tiles of
1024 or 2048 records: totals at and past each change of width, sessions at and
past a tile, weights and footprints in some sessions only, and a session with
a width of its own (then every session takes the default), against the oracle."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu
RTOL = 1e-5
CFG = dict(log2_slots=16, e_min=-2, kappa=0.0, normal_bins_log2=0)


def _records(n, seed, weighted, footprint):
    rng = np.random.default_rng(seed)
    p = rng.uniform(-2.0, 2.0, (3, n))
    run = np.arange(n) // 5 * 5  # five neighbouring records share a vertex: runs across wave and tile ends
    nrm = rng.normal(size=(3, n))
    v = rng.exponential(size=(3, n))
    v[1, rng.random(n) < 0.01] = np.nan
    extra = {}
    if weighted:
        extra["weight"] = rng.uniform(0.25, 2.0, n)
    if footprint:
        extra["footprint"] = rng.uniform(0.1, 1.0, n)
    return records(n, px=p[0, run], py=p[1, run], pz=p[2, run], nx=nrm[0, run], ny=nrm[1, run], nz=nrm[2, run],
                   r=v[0], g=v[1], b=v[2], **extra)


@pytest.mark.parametrize("sizes,extras,given", [
    ((1, 1023, 1024, 1025, 2049), "", False),
    ((1000, 3000, 5000), "weight", False),
    ((1000, 3000, 5000), "footprint", False),
    ((1000, 3000, 5000), "both", False),
    ((3000, 1025, 700), "", True),
    ((262144, 262144), "", False),        # the most records of tiles of 1024
    ((262144, 262145), "both", False),    # tiles of 2048
    ((1048576 - 5, 5, 1), "", False),     # tiles of 4096
])
def test_small_batches_match_the_oracle(sizes, extras, given):
    import oracle
    from paper_2005_07547_amd import psf
    weighted = [extras in ("weight", "both") and k % 2 == 0 for k in range(len(sizes))]
    footprint = [extras in ("footprint", "both") and k > 0 for k in range(len(sizes))]
    cfgs = [dict(CFG, weighted=w) for w in weighted]
    tabs = [psf.Table(**c, max_batch=n, **({"bin_per": 8} if given and k == 1 else {}))
            for k, (c, n) in enumerate(zip(cfgs, sizes))]
    orcs = [oracle.Oracle(**c) for c in cfgs]
    batch = psf.Batch(len(sizes))
    for it in range(2):
        recs = [_records(n, 100 * it + k, weighted[k], footprint[k]) for k, n in enumerate(sizes)]
        dev = [to_device(r) for r in recs]
        for (o, f), orc, rec in zip(batch.iterate(tabs, dev), orcs, recs):
            orc.insert(rec)
            orc.update()
            want, hit = orc.query(rec)
            assert np.array_equal(f.cpu().numpy(), hit)
            err = np.abs(o.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-30)
            assert float(err[:, hit.astype(bool)].max(initial=0.0)) <= RTOL
    for t, orc, w in zip(tabs, orcs, weighted):
        ex, cells = t.export(), orc.export()
        assert np.array_equal(ex["keys"], cells["keys"])
        assert w or np.array_equal(ex["c_old"].astype(np.uint64), cells["c_old"])
        assert t.stats()["dropped"] == 0
    batch.close()
