"""Every kernel in the sources has a name in the profile summariser (symbols as
the profiler prints them), so that no kernel's time drops out of a summary."""
import glob
import os
import re

import pytest

from paper_1805_05278_amd import build
from paper_1805_05278_amd import rocprof_summary as rs

SYMBOLS = {
    "k_axpy_cols": ("miqr::k_axpy_cols(long)", "axpy_cols"),
    "k_batch_reset": ("miqr::k_batch_reset(int*)", "batched_queue_reset"),
    "k_batched_blk": ("void miqr::k_batched_blk<1, 3>(miqr::BatchHeader const*)", "batched_blk_fp32"),
    "k_batched_ls": ("miqr::k_batched_ls(miqr::BatchHeader const*, int*, int*)", "batched_ls"),
    "k_batched_refine": ("miqr::k_batched_refine(miqr::BatchHeader const*, int)", "batched_refine"),
    "k_column_sumsq": ("miqr::k_column_sumsq(long)", "column_sumsq"),
    "k_copy_diagonal_blocks": ("miqr::k_copy_diagonal_blocks(long, long)", "copy_diagonal_blocks"),
    "k_copy_matrix": ("miqr::k_copy_matrix(long, long)", "copy_matrix"),
    "k_find_zero_diag": ("miqr::k_find_zero_diag(long)", "find_zero_diag"),
    "k_gemm": ("void miqr::k_gemm<128, 128, true, false, 1, 256>(miqr::GemmArgs)", "gemm_f32"),
    "k_gemm_bf16": ("void miqr::k_gemm_bf16<64, 64, true, false>(miqr::GemmArgs)", "gemm_bf16"),
    "k_normalize_r": ("miqr::k_normalize_r(long)", "normalize_r"),
    "k_scale_columns": ("miqr::k_scale_columns(long)", "scale_columns"),
    "k_set_identity": ("miqr::k_set_identity(long)", "set_identity"),
    "k_splitk_reduce": ("miqr::k_splitk_reduce(double const*, int)", "gemm_splitk_reduce"),
    "k_square_last_column": ("miqr::k_square_last_column(long)", "square_last_column"),
    "k_thin_nn": ("void miqr::k_thin_nn<4, 2>(miqr::ThinArgs)", "gemm_f64"),
    "k_thin_tn": ("void miqr::k_thin_tn<8>(miqr::ThinArgs)", "gemm_f64"),
    "k_trsm_diag": ("void miqr::k_trsm_diag<true>(int, long)", "trsm_diag"),
    "k_tsqr_down": ("void miqr::k_tsqr_down<true>(miqr::DownArgs)", "tsqr_down_leaf"),
    "k_tsqr_hr": ("miqr::k_tsqr_hr(miqr::HRArgs)", "tsqr_hr_root"),
    "k_tsqr_leaf": ("void miqr::k_tsqr_leaf<4>(miqr::ChainQRArgs)", "tsqr_chain_qr_leaf"),
    "k_tsqr_tree": ("void miqr::k_tsqr_tree<true>(miqr::ChainQRArgs)", "tsqr_chain_qr_tree"),
    "k_xpby_cols": ("miqr::k_xpby_cols(long)", "xpby_cols"),
    "k_zero_block_lower": ("miqr::k_zero_block_lower(long)", "zero_block_lower"),
}


def test_every_kernel_listed():
    found = set()
    for path in glob.glob(os.path.join(build.CSRC, "*.hip")):
        with open(path) as f:
            for m in re.finditer(r"__global__[^{;]*?\bvoid\b[^{;]*?(k_\w+)\s*\(|\n\s*void (k_\w+)\(",
                                 f.read()):
                found.add(m.group(1) or m.group(2))
    assert found == set(SYMBOLS)


@pytest.mark.parametrize("kernel", sorted(SYMBOLS))
def test_kernel_name(kernel):
    symbol, name = SYMBOLS[kernel]
    assert rs.library_name(symbol) == name
