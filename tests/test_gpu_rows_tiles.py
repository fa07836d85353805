"""Decode GEMMs of 33 and more rows by the column tiles that a workgroup owns: up to four run with 8 waves, five and six with
4.  The down projection of the 1024 wide shape has 65 k-tiles, which fill every wave's ring at least twice and leave some waves a
remainder, so that the loop over whole rings, its refills and its drain all run (test_routes.py checks that without a GPU)."""
import pytest

import test_gpu_rows as rows

pytestmark = pytest.mark.gpu

DOWN_MIN_WGS = {1: 128, 2: 64, 3: 44, 4: 32, 5: 26, 6: 22}  # column tiles of the down projection (64 of them) -> gemm_min_workgroups


@pytest.mark.parametrize("min_wgs", [8])  # residual GEMMs, 8 column tiles over 4 CUs; contractions shorter than two rings
def test_two_column_tiles_per_workgroup(min_wgs):
    rows.test_full_depth_step_over_a_given_number_of_rows("d128", min_wgs)


@pytest.mark.parametrize("tiles", list(DOWN_MIN_WGS))
def test_column_tiles_over_contractions_of_several_rings(tiles):
    rows.test_full_depth_step_over_a_given_number_of_rows("d1024", DOWN_MIN_WGS[tiles])
