"""The SH payload's binned insert in every tile the binning pass takes, with and
without weights and footprints, the run table read in place and transposed,
fused and as separate calls, with a remainder in the last tile, against the
binary64 oracle."""
import numpy as np
import pytest

from tests.helpers import to_device
from tests.test_gpu_sh import _compare, _oracle
from tests.test_gpu_sh_partitioned import _frame, env  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

# Every tile of the binning pass: 1024 records (few partitions), 2048 (1024 of
# them), 4096 (a width of its own, or more partitions)
TILES = {1024: dict(log2_slots=16), 2048: dict(log2_slots=18, part_log2=8), 4096: dict(log2_slots=16, bin_per=8),
         "4096-many-partitions": dict(log2_slots=19, part_log2=8)}


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("weighted,footprint", [(0, False), (0, True), (1, False), (1, True)])
@pytest.mark.parametrize("tile", list(TILES))
def test_every_binning_tile_matches_the_oracle(env, tile, weighted, footprint, transposed):
    torch, psf = env
    flags = psf.PSF_FLAG_TRANSPOSE_RUNS if transposed else 0
    t = orc = None
    for it, n in enumerate((8191, 4097)):  # one short of the last tile, and one over
        wl, rec = _frame(it, n, bool(weighted), footprint)
        rec["b"][2::19] = np.nan
        if t is None:
            cfg = dict(wl["table"], normal_bins_log2=0, payload=1, weighted=weighted, max_probe=256, **{
                k: v for k, v in TILES[tile].items() if k != "bin_per"})
            t, orc = psf.Table(**cfg, bin_per=TILES[tile].get("bin_per", 0), flags=flags), _oracle(cfg)
        if it == 0:
            t.iterate(to_device(rec))
        else:
            t.insert(to_device(rec))
            t.update()
        orc.insert(rec)
        orc.update()
    _compare(psf, t, orc, rec)
    assert t.stats()["dropped"] == 0
