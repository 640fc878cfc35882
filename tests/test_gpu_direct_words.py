"""The direct insert's leader election and word-wise adds: every record of a
wave in one cell, in cells of its own, and in a few interleaved cells; blocks
with a remainder; rejected records between; weighted and variance tables;
keys that find no slot.  Counters exact, sums against binary64."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 256, 257, 5000])
@pytest.mark.parametrize("cells", [1, 7, 64, 5000])
@pytest.mark.parametrize("kind", ["plain", "weighted", "variance"])
def test_direct_insert_matches_the_oracle(n, cells, kind):
    import oracle
    from paper_2005_07547_amd import psf
    rng = np.random.default_rng(n * 31 + cells)
    cell = rng.integers(0, cells, n)
    v = rng.exponential(size=(3, n))
    v[0, rng.random(n) < 0.05] = np.inf
    rec = records(n, px=cell % 50 + 0.5, py=cell // 50 + 0.5, pz=0.5, r=v[0], g=v[1], b=v[2])
    if kind == "weighted":
        rec["weight"] = rng.choice([0.0, 0.25, 1.5, np.nan], n, p=[0.1, 0.4, 0.4, 0.1]).astype(np.float32)
    cfg = dict(log2_slots=14, e_min=0, kappa=0.0, weighted=int(kind == "weighted"))
    t = psf.Table(**cfg, insert_mode=1, flags=psf.PSF_FLAG_TRACK_VARIANCE if kind == "variance" else 0)
    orc = oracle.Oracle(**cfg)
    for _ in range(2):
        t.insert(to_device(rec))
        orc.insert(rec)
    t.update()
    orc.update()
    ex, want = t.export(), orc.export()
    assert np.array_equal(ex["keys"], want["keys"])
    if kind == "weighted":  # sums of few binary fractions: exact in binary32
        assert np.array_equal(ex["c_old"].astype(np.float64), want["c_old"])
    else:
        assert np.array_equal(ex["c_old"].astype(np.uint64), want["c_old"])
    # binary32 sums of at most 2 n positive terms: within 2 n half units of the last place
    assert np.all(np.abs(ex["L"] - want["L"]) <= (2 * n + 4) * 2.0 ** -24 * np.abs(want["L"]))
    st = t.stats()
    assert st["dropped"] == 0 and st["skipped"] == orc.counters()["skipped"]


def test_direct_insert_counts_dropped_records():
    from paper_2005_07547_amd import psf
    n = 4096
    cell = np.arange(n) // 3
    rec = records(n, px=cell % 50 + 0.5, py=cell // 50 + 0.5)
    t = psf.Table(log2_slots=9, e_min=0, kappa=0.0, insert_mode=1, max_probe=512)
    t.insert(to_device(rec))
    t.update()
    ex, st = t.export(), t.stats()
    assert len(ex["keys"]) == 512 and st["dropped"] > 0
    assert int(ex["c_old"].sum()) + st["dropped"] == n
