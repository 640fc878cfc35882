"""Lookups where the roughness decides a lane at a time whether a vertex's
direction counts: waves of diffuse vertices, of glossy ones and mixed, with
directions at diffuse vertices that no key may see, thresholds that no vertex
and that every vertex passes, and sizes about a block's, against the oracle."""
import numpy as np
import pytest

from tests.helpers import records, to_device

pytestmark = pytest.mark.gpu
RTOL = 1e-5


def _vertices(n, thr, seed):
    rng = np.random.default_rng(seed)
    p, nrm, o = rng.uniform(-2, 2, (3, n)), rng.normal(size=(3, n)), rng.normal(size=(3, n))
    # stretches of 64 diffuse, 64 glossy and 64 mixed vertices
    kind = np.arange(n) // 64 % 3
    rough = np.where(kind == 0, 0.9, np.where(kind == 1, 0.1, rng.uniform(0.0, 1.0, n))).astype(np.float32)
    rough[rng.random(n) < 0.01] = np.nan
    diffuse = ~(rough < np.float32(thr))
    o[0, diffuse & (rng.random(n) < 0.5)] = np.nan
    o[1, diffuse & (rng.random(n) < 0.2)] = np.inf
    o[:, ~diffuse & (rng.random(n) < 0.02)] = np.nan  # no key
    v = rng.exponential(size=(3, n))
    return records(n, px=p[0], py=p[1], pz=p[2], nx=nrm[0], ny=nrm[1], nz=nrm[2], ox=o[0], oy=o[1], oz=o[2],
                   rough=rough, r=v[0], g=v[1], b=v[2])


@pytest.mark.parametrize("thr", [0.0, 0.3, float("inf")])
@pytest.mark.parametrize("n", [1, 255, 257, 4099])
def test_lookups_match_the_oracle(n, thr):
    import oracle
    from paper_2005_07547_amd import psf
    cfg = dict(log2_slots=16, e_min=0, kappa=0.0, max_level=3, rough_thr=thr)
    t, orc = psf.Table(**cfg), oracle.Oracle(**cfg)
    rec = _vertices(n, thr, 5)
    t.iterate(to_device(rec))
    orc.insert(rec)
    orc.update()
    for seed in (5, 6):  # the inserted vertices, and others
        q = _vertices(n, thr, seed)
        want, hit = orc.query(q)
        for out, found in (t.query(to_device(q)), t.query_levels(to_device(q), 0)):
            assert np.array_equal(found.cpu().numpy(), hit)
            err = np.abs(out.cpu().numpy() - want) / np.maximum(np.abs(want), 1e-30)
            assert float(err[:, hit.astype(bool)].max(initial=0.0)) <= RTOL
