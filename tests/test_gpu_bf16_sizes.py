"""bf16 contraction kernels on image sizes, batches and channel counts away from the workloads', against the oracle (the
checks of test_gpu_kernels)."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

CASES = [
    # n, B, H, W, Cin, Cout, k, stride, pad
    (1, 3, 28, 28, 32, 96, 3, 1, 1),     # nine rows of 28 pixels per tile, images that end inside a tile
    (2, 5, 7, 7, 64, 64, 3, 1, 1),       # several images per tile, the last tile ragged
    (1, 4, 14, 14, 40, 160, 3, 1, 1),    # 96-wide column blocks, a ragged channel chunk
    (1, 2, 24, 24, 32, 128, 3, 1, 1),    # ten rows of 24
    (2, 2, 15, 15, 32, 200, 3, 1, 1),    # 128-pixel tiles (few workgroups), two column blocks
    (1, 3, 12, 12, 48, 64, 5, 1, 2),     # padded 5 x 5
    (1, 4, 12, 12, 64, 64, 5, 1, 0),     # 5 x 5 without padding: output smaller than the input
    (2, 3, 28, 28, 128, 128, 3, 2, 1),   # stride 2 with the patch in LDS, nine rows of 14
    (1, 2, 20, 40, 64, 64, 3, 1, 1),     # rows of 40: six per tile
    (1, 2, 9, 100, 32, 32, 3, 1, 1),     # two rows of 100: a patch too wide for LDS, the gather kernels
    (3, 3, 16, 8, 96, 192, 3, 1, 1),     # not square
    (2, 3, 16, 16, 50, 64, 3, 1, 1),     # even channel counts that are no multiple of 8: dword loads, pairs of channels
    (1, 4, 12, 12, 33, 47, 3, 1, 1),     # odd counts: 16-bit loads, results straight from the accumulators
    (1, 2, 14, 14, 160, 50, 3, 1, 1),    # 50 outputs of whole-vector input, two 64-wide blocks back
    (1, 3, 15, 15, 16, 19, 3, 1, 1),     # one tile of channels in the weight gradient, mostly padding
    (2, 2, 12, 12, 17, 300, 3, 1, 1),    # 300 outputs: three wide blocks; backward over a ragged last chunk of 300
    (1, 2, 10, 10, 18, 130, 5, 1, 2),    # 5 x 5: two groups of taps per window row in the weight gradient
    (1, 2, 9, 9, 17, 20, 7, 1, 3),       # 7 x 7, odd count
    (1, 3, 16, 16, 50, 94, 3, 2, 1),     # stride 2: even and odd columns of the input in the weight gradient
    (1, 3, 11, 13, 21, 23, 3, 2, 1),     # same, odd everything
]


@pytest.mark.parametrize("case", CASES)
def test_odd_sizes_match_oracle(gpu, case):
    tk.test_conv_kernels_match_oracle(gpu, case, 1)


@pytest.mark.parametrize("case", [(2, 5, 28, 28, 32, 64, 3, 1, 1), (1, 7, 7, 7, 64, 128, 3, 1, 1), (2, 3, 28, 28, 128, 128, 3, 2, 1)])
def test_column_sums_on_odd_sizes(gpu, case):
    """The column sums a convolution leaves, added over its partial rows, are those of what it stored."""
    import numpy as np
    torch, pb = gpu
    n, B, H, W, Cin, Cout, k, stride, pad = case
    rng = np.random.default_rng(11)
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    x = tk.upload(torch, tk.to_bf16_grid(rng.standard_normal((n, B, H, W, Cin))), 1)
    w = tk.upload(torch, tk.to_bf16_grid(rng.standard_normal((n, Cout, k, k, Cin)) / np.sqrt(k * k * Cin)), 1)
    y = torch.zeros((n, B, Ho, Wo, Cout), dtype=torch.bfloat16, device="cuda")
    partial = torch.full((n * 1024 * 2 * Cout,), float("nan"), dtype=torch.float64, device="cuda")
    S = pb.parle_k_conv_forward_colsums(pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, k, stride, pad), x, w, None, y, partial, 1024)
    torch.cuda.synchronize()
    assert S > 0
    got = partial[:n * S * 2 * Cout].cpu().numpy().reshape(n, S, 2, Cout).sum(axis=1)
    yv = y.double().cpu().numpy().reshape(n, B * Ho * Wo, Cout)
    assert np.max(np.abs(got[:, 0] - yv.sum(axis=1)) / np.abs(yv).sum(axis=1)) < 1e-5
    assert np.max(np.abs(got[:, 1] / (yv * yv).sum(axis=1) - 1)) < 1e-5
