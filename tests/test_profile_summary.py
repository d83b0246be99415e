"""Every layer kernel's name, as rocprofv3 prints it, falls into the class that pc_profile_read counts it in."""
import pytest

from paper_2406_00766_amd.profile_summary import kernel_class


@pytest.mark.parametrize("name,cls", [
    ("void pc::k_flow<4, 2, 1, false, true>(float const*)", "sum_fwd"),
    ("pc::k_flow<8, 2, 2, true, false>", "sum_bwd_child"),
    ("pc::k_sum_16<false, 4>", "sum_fwd"),
    ("pc::k_sum_16<true, 1>", "sum_bwd_child"),
    ("pc::k_sum_mfma<64, 1, 4, true, false, 1>", "sum_bwd_child"),
    ("pc::k_sum_mfma<32, 1, 4, false, false, 3>", "sum_fwd"),
    ("pc::k_sum_merge", "sum_fwd"),
    ("pc::k_param_flow_16", "sum_bwd_param"),
    ("pc::k_prod_fwd<2, 4, 2, 8, double, false>", "prod_fwd"),
    ("pc::k_em_theta<4, 1, false>", "em"),
    ("pc::k_em_row_sums<4>", "em"),
    ("pc::k_begin_forward", "misc"),
])
def test_kernel_class(name, cls):
    assert kernel_class(name) == cls


@pytest.mark.parametrize("name,cls", [
    ("void pc::k_chain<false>(float const*, float*)", "sum_fwd"),
    ("pc::k_chain<true>", "sum_bwd_child"),
    ("pc::k_sum_16<true, 1, 1>", "sum_bwd_child"),
    ("pc::k_prod_tile<16, 4>", "prod_fwd"),
    ("pc::k_class_bwd<2, 8, 16>", "prod_bwd"),
    ("pc::k_begin_forward<0>", "misc"),
    ("pc::k_begin_forward<32>", "input_fwd"),
])
def test_kernel_class_of_chains_tiles_and_begins(name, cls):
    assert kernel_class(name) == cls
