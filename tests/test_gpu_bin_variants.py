"""Every instantiation of the RGB binning pass: each tile it takes, with and
without footprints and weights, with the variance's squared sums, alone and
batched, over whole tiles and a remainder, against the oracle."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu
RTOL = 1e-5
# tiles of 1024 records need at most 512 partitions, of 2048 at most 1024; the
# others are binning widths
TILES = {1024: dict(log2_slots=16), 2048: dict(log2_slots=18, part_log2=8), 4096: dict(log2_slots=16, bin_per=8),
         6144: dict(log2_slots=16, bin_per=12), 8192: dict(log2_slots=16, bin_per=16)}
CFG = dict(e_min=-2, kappa=0.0, normal_bins_log2=1, max_level=3, rough_thr=0.3)


def _records(n, seed, weighted, footprint):
    rng = np.random.default_rng(seed)
    p = rng.uniform(-2.0, 2.0, (3, n))
    run = np.arange(n) // 5 * 5
    nrm, o, v = rng.normal(size=(3, n)), rng.normal(size=(3, n)), rng.exponential(size=(3, n))
    v[1, rng.random(n) < 0.01] = np.nan
    extra = {}
    if weighted:
        extra["weight"] = np.where(rng.random(n) < 0.1, 0.0, rng.uniform(0.25, 2.0, n))
    if footprint:
        extra["footprint"] = rng.uniform(0.3, 1.2, n)[run]
    return records(n, px=p[0, run], py=p[1, run], pz=p[2, run], nx=nrm[0, run], ny=nrm[1, run], nz=nrm[2, run],
                   ox=o[0, run], oy=o[1, run], oz=o[2, run], rough=rng.uniform(0.0, 1.0, n)[run],
                   r=v[0], g=v[1], b=v[2], **extra)


def _close(out, found, orc, rec):
    want, hit = orc.query(rec)
    assert np.array_equal(found.cpu().numpy(), hit)
    err = np.abs(out.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-30)
    assert float(err[:, hit.astype(bool)].max(initial=0.0)) <= RTOL


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("kind", ["plain", "footprint", "weighted", "both", "variance"])
@pytest.mark.parametrize("tile", list(TILES))
def test_binning_matches_the_oracle(tile, kind, batched):
    import oracle
    from paper_2005_07547_amd import psf
    weighted, footprint = kind in ("weighted", "both"), kind in ("footprint", "both")
    flags = psf.PSF_FLAG_TRACK_VARIANCE if kind == "variance" else 0
    slots = {k: v for k, v in TILES[tile].items() if k == "log2_slots"}
    sizes = (2 * 8192 + 77, 6145) if batched else (2 * 8192 + 77,)
    # (a batch's second session carries no footprints)
    carried = [(weighted, footprint), (weighted, False)]
    tabs = [psf.Table(**CFG, **TILES[tile], weighted=int(weighted), flags=flags) for _ in sizes]
    orcs = [oracle.Oracle(**CFG, **slots, weighted=int(weighted)) for _ in sizes]
    batch = psf.Batch(len(sizes))
    for it in range(2):
        recs = [_records(n, 10 * it + k, *carried[k]) for k, n in enumerate(sizes)]
        dev = [to_device(r) for r in recs]
        answers = batch.iterate(tabs, dev) if batched else [tabs[0].iterate(dev[0])]
        for (out, found), orc, rec in zip(answers, orcs, recs):
            orc.insert(rec)
            orc.update()
            _close(out, found, orc, rec)
    for t, orc in zip(tabs, orcs):
        st, ex, o = t.stats(), t.export(), orc.export()
        assert st["dropped"] == 0 and st["skipped"] == orc.counters()["skipped"]
        assert np.array_equal(ex["keys"], o["keys"])
        assert np.allclose(ex["c_old"].astype(np.float64), o["c_old"], rtol=1e-6 if weighted else 0)
        if kind == "variance":
            keys, var = t.export_variance()
            o_keys, o_var = orc.export_variance()
            m = o["L"][0] * 0.25 + o["L"][1] * 0.5 + o["L"][2] * 0.25
            assert np.array_equal(keys, o_keys)
            assert np.all(np.abs(var - o_var) <= RTOL * (o_var + m * m) + 1e-30)
    batch.close()
