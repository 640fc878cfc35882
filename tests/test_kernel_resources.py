"""What the compiler recorded of the built library's kernels: registers kept
out of scratch memory, and dynamic LDS that starts where its widest accesses
need it."""
import os

import pytest

from paper_2005_07547_amd import build


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.OUT):
        build.build()
    return build.kernel_resources()


def test_every_kernel_family_is_in_the_library(kernels):
    for part in ("k_bin", "k_bin_batch", "k_merge", "k_merge_batch", "k_merge_sh", "k_unstage", "k_query",
                 "k_insert_direct", "k_estimate", "k_sample_paths"):
        assert any(f"{len(part)}{part}" in n for n in kernels), part


def test_no_binning_kernel_spills_to_scratch(kernels):
    spilled = [n for n, k in kernels.items() if "k_bin" in n and (k["private_segment_fixed_size"] or k["vgpr_spill_count"])]
    assert not spilled


def test_binning_lds_starts_at_a_multiple_of_16(kernels):
    # keys are staged there as 8-byte words, values as 16-byte ones; the
    # dynamic part starts where the static part ends
    odd = {n: k["group_segment_fixed_size"] for n, k in kernels.items() if "k_bin" in n and k["group_segment_fixed_size"] % 16}
    assert not odd


def test_check_refuses_scratch_and_odd_lds():
    good = {"private_segment_fixed_size": 0, "vgpr_spill_count": 0, "group_segment_fixed_size": 592}
    build.check_resources({"5k_bin": good})
    for bad in ({"private_segment_fixed_size": 4}, {"vgpr_spill_count": 1}, {"group_segment_fixed_size": 68}):
        with pytest.raises(RuntimeError):
            build.check_resources({"5k_bin": dict(good, **bad)})
    with pytest.raises(RuntimeError):
        build.check_resources({"7k_merge": good})
