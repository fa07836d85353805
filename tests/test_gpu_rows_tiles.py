"""Decode GEMMs of 33 and more rows by the column tiles that a workgroup owns: up to four run with 8 waves, five and six with
4.  The widths and workgroup targets of test_gpu_rows.py give one, three, four, five and six; this one adds two."""
import pytest

import test_gpu_rows as rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("min_wgs", [8])  # residual GEMMs, 8 column tiles over 4 CUs
def test_two_column_tiles_per_workgroup(min_wgs):
    rows.test_full_depth_step_over_a_given_number_of_rows("d128", min_wgs)
