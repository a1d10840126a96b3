"""fp32 contraction kernels at the sizes where their tiles, splits and dispatch rules have edges, against the oracle's
convolution (the checks of test_gpu_kernels: forward with and without epilogue, input gradient plain and masked onto an
existing gradient, weight gradient, bias gradient)."""
import numpy as np
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


CONV_CASES = [
    # n, B, H, W, Cin, Cout, k, stride, pad
    (1, 1, 3, 3, 8, 1, 3, 1, 1),         # the fewest channels the split kernel takes, one output channel
    (2, 5, 7, 7, 24, 36, 3, 1, 1),       # tiles that run over several images, the last one ragged
    (1, 3, 28, 28, 16, 64, 3, 1, 1),     # nine rows of 28 pixels per tile, images that end inside a tile
    (2, 2, 24, 24, 20, 32, 3, 1, 1),     # ten rows of 24
    (1, 4, 15, 15, 33, 47, 3, 1, 1),     # odd channel counts: dword loads, results straight from the accumulators
    (1, 3, 14, 14, 50, 20, 3, 1, 1),     # even channel counts: 8-byte loads
    (1, 2, 9, 130, 12, 16, 3, 1, 1),     # one row per tile, 17 strips of eight columns
    (1, 1, 5, 300, 12, 8, 3, 1, 1),      # rows wider than a tile: the gather kernels
    (2, 3, 12, 12, 20, 52, 5, 1, 0),     # 5 x 5 without padding
    (1, 2, 10, 11, 16, 130, 5, 1, 2),    # padded 5 x 5, three 64-wide column blocks
    (1, 2, 9, 9, 16, 24, 7, 1, 3),       # 7 x 7: three groups of taps per window row
    (1, 3, 8, 8, 24, 40, 2, 1, 0),       # 2 x 2
    (2, 3, 11, 9, 16, 48, 3, 2, 1),      # stride 2, odd extents
    (2, 5, 16, 16, 36, 20, 3, 2, 1),     # stride 2, two images per tile, odd batch
    (1, 2, 28, 28, 12, 33, 5, 2, 2),     # stride 2 under a 5 x 5 window
    (1, 70, 8, 8, 64, 320, 3, 1, 1),     # 320 outputs
]


@pytest.mark.parametrize("case", CONV_CASES)
def test_split_convolutions_match_oracle(gpu, case):
    tk.test_conv_kernels_match_oracle(gpu, case, 0)


WINDOW_CASES = [
    # n, B, H, W, Cin, Cout, k, stride, pad: backward-data with an image per workgroup, 128 columns of products at a time
    (1, 1, 2, 2, 1, 1, 2, 1, 0),         # one output pixel, one channel
    (2, 3, 9, 9, 32, 64, 2, 1, 0),       # 128 columns exactly, all 64 pixels and contraction values
    (1, 2, 6, 6, 33, 17, 2, 1, 0),       # 132 columns: a second chunk of four
    (1, 2, 5, 12, 132, 16, 2, 1, 0),     # a tap wider than a chunk
    (1, 2, 6, 6, 131, 33, 2, 1, 0),      # the same, odd
    (2, 2, 7, 7, 28, 48, 3, 1, 1),       # two chunks, the second nearly full, taps across the seam
    (1, 3, 4, 8, 15, 63, 3, 1, 1),       # 32 output pixels: one row tile
    (1, 3, 3, 11, 15, 20, 3, 1, 1),      # 33
    (3, 2, 10, 10, 7, 50, 7, 1, 2),      # 7 x 7
    (1, 1, 12, 12, 4, 3, 5, 1, 0),       # a single vector per pixel
    (2, 2, 8, 8, 50, 40, 3, 1, 1),       # even counts: two channels at a time, four chunks, taps across every seam
    (1, 2, 6, 6, 2, 17, 2, 1, 0),        # ... a single pair
    (1, 2, 5, 12, 130, 33, 2, 1, 0),     # ... a tap wider than a chunk
    (2, 2, 7, 7, 54, 9, 3, 1, 1),        # the widest tap of a 3 x 3 window with few outputs
    (2, 2, 7, 7, 56, 32, 3, 1, 1),       # ... and the first that takes the row kernel
]


@pytest.mark.parametrize("case", WINDOW_CASES)
def test_window_products_match_oracle(gpu, case):
    tk.test_conv_kernels_match_oracle(gpu, case, 0)


@pytest.mark.parametrize("case", [(1, 3, 8, 8, 32, 96, 3, 1, 1), (1, 2, 12, 12, 20, 50, 5, 1, 0), (1, 3, 16, 16, 16, 32, 3, 2, 1)])
def test_split_convolutions_keep_infinities_and_nan(gpu, case):
    """An infinite or NaN operand reaches the results it reaches in plain arithmetic, with the same sign, and no others:
    the corrections of the split, which are NaN there, stay out."""
    torch, pb = gpu
    n, B, H, W, Cin, Cout, k, stride, pad = case
    rng = np.random.default_rng(5)
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    x = rng.standard_normal((n, B, H, W, Cin)).astype(np.float32)
    w = (rng.standard_normal((n, Cout, k, k, Cin)) / np.sqrt(k * k * Cin)).astype(np.float32)
    dy = rng.standard_normal((n, B, Ho, Wo, Cout)).astype(np.float32)
    x[0, 0, 3, 4, 1], x[0, 1, 5, 2, 3], x[0, 1, 5, 3, 3] = np.inf, -np.inf, 5.0e37
    dy[0, 0, 1, 2, 5], dy[0, 1, 3, 3, 7] = np.inf, np.nan
    desc = pb.parle_conv_desc(0, n, B, H, W, Cin, Cout, k, stride, pad)
    dx_, dw_, ddy = (tk.upload(torch, a, 0) for a in (x, w, dy))
    y = torch.zeros((n, B, Ho, Wo, Cout), dtype=torch.float32, device="cuda")
    gx = torch.zeros((n, B, H, W, Cin), dtype=torch.float32, device="cuda")
    gw = torch.zeros((n, Cout, k, k, Cin), dtype=torch.float32, device="cuda")
    scratch = torch.zeros(max(pb.parle_k_conv_scratch_bytes(desc) // 4, 4), dtype=torch.float32, device="cuda")
    pb.parle_k_conv_forward(desc, dx_, dw_, None, None, 0, y)
    pb.parle_k_conv_backward_data(desc, ddy, dw_, None, 0, torch.zeros_like(dw_), gx)
    pb.parle_k_conv_backward_weight(desc, ddy, dx_, scratch, gw)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        ry, rdx, rdw = tk.oracle_conv(x[0], w[0], None, None, False, stride, pad, dy[0])
    for name, got, ref in (("forward", y, ry), ("input gradient", gx, rdx), ("weight gradient", gw, rdw)):
        got = tk.download(got[0])
        # a matrix product in the reference spreads an infinity over its zero padding as NaN only where one meets it
        fin = np.isfinite(ref)
        assert (np.isfinite(got) == fin).all(), name
        inf = np.isinf(ref)
        assert (got[inf] == ref[inf]).all(), name
        assert np.isnan(got[np.isnan(ref)]).all(), name
        tk.assert_near(name, got[fin], ref[fin], 1e-6, 2e-5 * np.abs(ref[fin]).max())


@pytest.mark.parametrize("arch", [
    dict(kind="lenet", H=28, W=28, C=1, c1=20, c2=72, k=5, fc=40, classes=10),   # products through memory
    dict(kind="lenet", H=28, W=28, C=1, c1=30, c2=72, k=5, fc=40, classes=10),   # directly
    dict(kind="allcnn", H=12, W=12, C=3, ca=16, cb=32, classes=10),              # directly, padded
])
def test_networks_choose_between_two_input_gradient_routes(gpu, monkeypatch, arch):
    import test_gpu_nets as tn
    monkeypatch.setitem(tn.SMALL, "route", tn.onets.arch(arch["kind"], **{k: v for k, v in arch.items() if k != "kind"}))
    tn.test_one_step_loss_and_gradient(gpu, "route", 0)
