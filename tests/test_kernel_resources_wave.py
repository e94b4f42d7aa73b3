"""Register and spill budgets of the kernels whose design rests on them beside the square
MHD tiles: the wide FP32 flux kernels, the dust passes, and the closure's convolutions and
gradients.  Read from the compiler's report for gfx950 (host only); a failure names the
budget that moved."""
import re

import pytest

from tests.test_kernel_resources import LDS_PER_CU, _resources


@pytest.fixture(scope="module")
def fused():
    return _resources("mhd_fused.hip")


@pytest.fixture(scope="module")
def dust():
    return _resources("dust_kernels.hip")


@pytest.fixture(scope="module")
def closure():
    return _resources("cnn.hip")


def _named(res, pattern, count):
    """The kernels whose mangled name matches, with the match: as many as are built."""
    hits = [(m, v) for n, v in res.items() for m in [re.match(pattern, n)] if m]
    assert len(hits) == count, (pattern, sorted(res))
    return hits


def test_wide_fp32_flux_kernels_run_four_waves(fused):
    for m, k in _named(fused, r"_ZN3mhd12k_flux3_wideILi(\d)ELi(\d)ELb\dEE", 12):
        assert k["Occupancy"] >= 4 and k["ScratchSize"] == 0, (m.group(0), k)


def test_dust_passes_keep_their_waves(dust):
    # mangled template arguments: <RECON, STAGE, real, rows, SOLO>
    for m, k in _named(dust, r"_ZN3mhd12k_fluid_passILi(\d)ELi(\d)E([df])Li(\d)ELb(\d)EE", 22):
        recon, real, rows, solo = m.group(1), m.group(3), m.group(4), m.group(5)
        least = (3 if real == "f" else 2) if recon == "1" else (4 if real == "f" else 3)
        if recon == "1" and real == "f" and rows == "1":
            least = 4
        if solo == "1":
            least = 2  # (all waves run at once at two per SIMD)
        assert k["Occupancy"] >= least and k["ScratchSize"] == 0, (m.group(0), least, k)
    for m, k in _named(dust, r"_ZN3mhd12k_donor_passILi(\d)EdE", 2):
        assert k["Occupancy"] >= 3 and k["ScratchSize"] == 0, (m.group(0), k)


def test_convolutions_hold_their_weights_in_registers(closure):
    # <input channels, MODE, rows and planes of a wave, groups of them along y and z>
    for m, k in _named(closure, r"_ZN3mhd6k_convILi(\d+)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)EE", 12):
        assert k["Occupancy"] >= 2 and k["LDS Size"] <= LDS_PER_CU, (m.group(0), k)
        # (32 rows of a plane stage 102 halo rows: a few loop-invariant dwords are reloaded)
        assert k["ScratchSize"] <= (16 if m.group(3) == "8" else 0), (m.group(0), k)
    for m, k in _named(closure, r"_ZN3mhd6k_gradILi(\d+)EE", 2):
        # nine waves, one workgroup per CU: three waves on a SIMD
        assert k["Occupancy"] >= 3 and k["ScratchSize"] == 0 and k["LDS Size"] <= LDS_PER_CU, (m.group(0), k)
