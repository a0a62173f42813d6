"""The counter summaries name a kernel as the library's launch log does, so that a record's traffic and occupancy are found."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1706_00095_amd"))

# a profiler's name, the launch log's
MATRIX = {
    "void cg::split_patch_kernel<3, 2, 4, 1, 4, false>(cg::IgemmProblem)": "igemm_patch_kernel<128x128,4>",
    "void cg::split_patch_kernel<3, 3, 1, 2, 5, true>(cg::IgemmProblem)": "igemm_patch16_kernel<48x128,5>",
    "void cg::split_patch_kernel<2, 1, 4, 1, 6, false>(cg::IgemmProblem)": "igemm_patch_kernel<64x128,6,bf16x3>",
    "void cg::split_patch_kernel<3, 3, 4, 1, 4, false, true>(cg::IgemmProblem)": "igemm_patch_kernel<192x128,4>",
    "void cg::stem_fwd_kernel<3, 2>(cg::StemArgs)": "igemm_stem_kernel<96>",
    "void cg::direct_kernel<2, 1>(cg::DirectArgs)": "igemm_direct_kernel<16x32,4c>",
    "void cg::split_wgrad_kernel<3, 2, 8>(cg::IgemmProblem)": "igemm_kernel<128x144,band8>",
    "void cg::split_gemm_kernel<3, 2, 4, cg::(anonymous namespace)::LoadA<2, 1>, cg::(anonymous namespace)::LoadBRows<2, true, false>, true>(cg::IgemmProblem)":
        "igemm_kernel<128x128,4rc,pieces>",
    "void cg::igemm_kernel<1, 4, 3, 1, 4, cg::(anonymous namespace)::KLoader4<96, 1>, cg::(anonymous namespace)::RowsLoader<128, true>, 0>(cg::IgemmProblem)":
        "igemm_kernel<96x128,4rc>",
}


@pytest.mark.parametrize("name", list(MATRIX), ids=lambda n: n[5:40])
def test_matrix_kernels(name):
    from pmc_mfma_busy import is_matrix_kernel
    from pmc_traffic import label
    assert label(name) == MATRIX[name] and is_matrix_kernel(name)


def test_others():
    from pmc_mfma_busy import is_matrix_kernel
    from pmc_traffic import label
    assert label("void cg::reduce_sgd_kernel<8, true>(cg::SgdArgs)") == "reduce_sgd_kernel<8,tree>"
    assert not is_matrix_kernel("void cg::(anonymous namespace)::splitk_finish_kernel<8, true, false>(cg::FinishArgs)")
    assert not is_matrix_kernel("void cg::reduce_sgd_kernel<8, true>(cg::SgdArgs)")
