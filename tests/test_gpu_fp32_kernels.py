"""fp32 contraction kernels at the sizes where their tiles, splits and dispatch rules have edges, against the oracle's
convolution (the checks of test_gpu_kernels: forward with and without epilogue, input gradient plain and masked onto an
existing gradient, weight gradient, bias gradient)."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

FC_CASES = [
    # n, B, H, W, Cin, Cout, k, stride, pad
    (1, 1, 1, 1, 1, 1, 1, 1, 0),        # one row, one value
    (2, 33, 1, 1, 33, 5, 1, 1, 0),      # rows that are no whole vectors, in every operand
    (2, 17, 1, 1, 260, 36, 1, 1, 0),    # 16-wide tiles, eight wavefronts over a contraction of nine ragged batches
    (3, 31, 1, 1, 257, 63, 1, 1, 0),    # same, odd everything
    (2, 1024, 1, 1, 40, 44, 1, 1, 0),   # the longest batch the weight gradient takes in one piece
    (1, 1025, 1, 1, 40, 44, 1, 1, 0),   # one row more: the generic kernel with split sums
    (6, 128, 1, 1, 96, 500, 1, 1, 0),   # 32-wide tiles, four wavefronts each, ragged last column tile
    (5, 128, 1, 1, 64, 1060, 1, 1, 0),  # more than two tiles per compute unit: two tiles per workgroup, an odd number of them
    (2, 4, 7, 7, 50, 96, 1, 1, 0),      # a 1 x 1 convolution on 7 x 7 pixels
]


@pytest.mark.parametrize("case", FC_CASES)
def test_plain_products_match_oracle(gpu, case):
    tk.test_conv_kernels_match_oracle(gpu, case, 0)
