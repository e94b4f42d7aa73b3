"""The benchmark's bytes per cell of each MHD kernel against the fields the kernels hold:
FP64 words throughout, or FP32 words with the total energy in FP64 (host only)."""
import pytest

import bench


@pytest.mark.parametrize("word,table", [(8, bench.KERNEL_ALGO), (4, bench.KERNEL_ALGO_FP32)])
def test_kernel_bytes_add_up_from_the_fields(word, table):
    cells = 4 * word + 8  # density, three momenta; the energy in FP64 in both forms
    faces = 3 * word      # the face fields
    edge = 9 * word + 1   # two face values of E per direction, the cell's E, the flow codes
    assert table["mhd_flux_update_predictor"]["bytes"] == cells + faces + cells + edge
    assert table["mhd_flux_update_corrector"]["bytes"] == cells + faces + 2 * cells + edge
    assert table["mhd_ct_predictor"]["bytes"] == edge + 2 * faces
    assert table["mhd_ct_corrector"]["bytes"] == edge + 2 * faces + cells
    assert table["cfl"]["bytes"] == cells + faces
