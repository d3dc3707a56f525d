"""Kernel families of the steps' column passes: every form belongs to one (CPU)."""
import pytest

from paper_2303_01471_amd import profiling


@pytest.mark.parametrize("kernel,family", [
    ("void qhd::k_lf_col_tw<64>(qhd::InstDev const*, int const*, int, HIP_vector_type<float, 2u>*)", ("col_pass_2d_qaa_lf/n64", 20.0)),
    ("k_lf_col_tw<128>", ("col_pass_2d_qaa_lf/n128", 20.0)),
    ("k_lf_col_2d<256, 8>", ("col_pass_2d_qaa_lf/n256", 20.0)),
    ("k_col_axis_tw<128, 16, 0, false>", ("col_pass_2d/n128", 24.0)),
    ("k_col_axis_tw<64, 8, 1, true>", ("col_pass_2d_qaa/n64", 24.0)),
    ("k_col_axis_split<512, true>", ("col_pass_2d/n512", 24.0)),
    ("k_col_axis_2d<32, 8, 0, true>", ("col_pass_2d/n32", 24.0)),
    ("k_row_axis_2d<128, 16, 0, true>", ("row_pass_2d/n128", 24.0)),
])
def test_family(kernel, family):
    assert profiling.family_of(kernel) == family
