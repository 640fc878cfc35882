"""The SH payload's binned insert (the strategy a table takes by itself)
against the binary64 oracle: fused frames, inserts split into several calls
and over the staging capacity, partitions with more touched cells than one
round of sums holds, rejected samples, and the direct insert's results."""
import numpy as np
import pytest

from tests.helpers import take, to_device
from tests.test_gpu_sh import _compare, _oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_2005_07547_amd import psf
    psf.load()
    return torch, psf


def _frame(it, n=None, weighted=False, footprint=False):
    from synth import workloads as W
    wl = W.tiny(alpha_mode=W.ALPHA_PAPER)
    rec = dict(W.make_scene(wl).generate(wl["gen"], it))
    rec["rough"] = None
    if weighted:
        rec["weight"] = W.mis_weights(rec["px"].shape[0], seed=it)
    if footprint:
        rec["footprint"] = W.footprints(rec, wl, spread=1.5)
    return wl, (rec if n is None else take(rec, np.arange(n)))


# (slots, partition width): the default; narrow partitions; two partitions whose
# cells take several rounds of sums
TABLES = [(16, 0), (16, 8), (13, 12)]


@pytest.mark.parametrize("log2_slots,part_log2", TABLES)
@pytest.mark.parametrize("weighted,footprint", [(0, False), (1, True)])
def test_fused_frames_match_the_oracle(env, log2_slots, part_log2, weighted, footprint):
    torch, psf = env
    if weighted and part_log2 == 12:
        part_log2 = 11
    t = orc = None
    for it in range(3):
        # 8192 records, then one short of a binning tile, then a few
        wl, rec = _frame(it, (None, 4095, 5)[it], bool(weighted), footprint)
        if t is None:
            cfg = dict(wl["table"], normal_bins_log2=0, payload=1, log2_slots=log2_slots, part_log2=part_log2,
                       max_probe=1 << 12, weighted=weighted)
            t, orc = psf.Table(**cfg), _oracle(cfg)
        t.iterate(to_device(rec))
        orc.insert(rec)
        orc.update()
    _compare(psf, t, orc, rec)
    st = t.stats()
    assert st["dropped"] == 0 and st["updates"] == 3
    assert st["skipped"] == (0 if not weighted else sum(int((_frame(i, m, True)[1]["weight"] == 0).sum())
                                                        for i, m in ((0, None), (1, 4095), (2, 5))))


def test_separate_inserts_over_the_staging_capacity_match_the_oracle(env):
    torch, psf = env
    wl, a = _frame(0)
    _, b = _frame(1, 5001)
    cfg = dict(wl["table"], normal_bins_log2=0, payload=1, max_batch=4096)
    t, orc = psf.Table(**cfg), _oracle(cfg)
    for _ in range(2):
        for rec in (a, b):
            t.insert(to_device(rec))
            orc.insert(rec)
        t.update()
        orc.update()
    t.iterate(to_device(a))  # more records than one launch stages
    orc.insert(a)
    orc.update()
    _compare(psf, t, orc, a)


def test_rejected_samples_and_full_partitions_equal_the_direct_insert(env):
    torch, psf = env
    wl, rec = _frame(0)
    rec["px"][::7] = np.nan
    rec["g"][3::11] = np.inf
    # 1024 slots for several thousand cells: most keys find no slot
    stats = []
    for mode in (0, 1):
        t = psf.Table(**dict(wl["table"], normal_bins_log2=0, payload=1, log2_slots=10, max_probe=1 << 10,
                             insert_mode=mode))
        t.iterate(to_device(rec))
        ex, st = psf.export_sh(t), t.stats()
        assert len(ex["keys"]) == 1024 and int(ex["c_old"].sum()) == len(rec["px"]) - st["skipped"] - st["dropped"]
        stats.append({k: st[k] for k in ("submitted", "skipped", "coord_overflow", "occupied", "updates")})
    assert stats[0] == stats[1]
