"""Weight (and bias) gradients of 3x3 bf16 layers, nine taps per wavefront, stride 1 and 2: every arrangement of wavefronts,
both block shapes, one and several blocks per split, an odd batch of 8x8 images, against plain products in 64 bits."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

CASES = [
    # n, B, H, W, Cin, Cout, stride: dy tiles x x tiles per workgroup
    (2, 3, 16, 16, 64, 64, 1),     # 2 x 2
    (1, 7, 8, 8, 128, 64, 1),      # 2 x 2, two images per block, odd batch
    (3, 40, 32, 32, 64, 128, 1),   # 2 x 2, many splits
    (1, 5, 8, 32, 32, 64, 1),      # 2 x 1, one row of blocks
    (2, 9, 8, 8, 96, 64, 1),       # 2 x 1
    (1, 6, 24, 16, 96, 96, 1),     # 3 x 1
    (2, 5, 8, 8, 64, 96, 1),       # 3 x 1, odd batch
    (1, 4, 16, 16, 32, 128, 1),    # 4 x 1
    (1, 3, 8, 8, 96, 256, 1),      # 4 x 1, one block per split
    (1, 8, 16, 48, 64, 160, 1),    # 5 x 1, three blocks per row
    (1, 3, 8, 8, 32, 160, 1),      # 5 x 1
    (1, 5, 28, 28, 96, 96, 1),     # images that do not cut into blocks: two columns of blocks, the second with 12 pixels
    (2, 3, 14, 14, 64, 128, 1),    # 2 x 2, rows of 14
    (1, 65, 7, 7, 64, 64, 1),      # pairs of rows of 7, the last pair half beyond the image, odd batch
    (2, 57, 7, 8, 32, 160, 1),     # rows of 8
    (1, 3, 15, 15, 64, 64, 1),     # a row more than a block, 15 pixels
    (1, 4, 12, 12, 32, 128, 1),    # 4 x 1
    (1, 2, 9, 40, 64, 64, 1),      # three columns of blocks
    (1, 2, 16, 128, 64, 64, 1),    # eight columns of blocks
    (2, 3, 32, 32, 32, 64, 2),     # stride 2: two dy tiles, rows of 16
    (1, 5, 16, 16, 64, 64, 2),     # 8x8 results, odd batch
    (1, 6, 8, 64, 64, 96, 2),      # three, one row of blocks, two per row
    (2, 3, 16, 16, 32, 96, 2),
    (3, 40, 32, 32, 64, 128, 2),   # four, many splits
    (1, 1, 16, 16, 96, 128, 2),    # one block
    (1, 3, 32, 96, 32, 160, 2),    # five
    (1, 4, 16, 16, 32, 160, 2),
]


@pytest.mark.parametrize("case", CASES)
def test_weight_and_bias_gradient(gpu, case):
    torch, pb = gpu
    n, B, H, W, Cin, Cout, stride = case
    P, Q = H // stride, W // stride
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn((n, B, H, W, Cin), generator=gen, device="cuda").bfloat16()
    dy = torch.randn((n, B, P, Q, Cout), generator=gen, device="cuda").bfloat16()
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, 3, stride, 1)
    scratch = torch.empty(max(pb.parle_k_conv_scratch_bytes(desc), 256), dtype=torch.uint8, device="cuda")
    wsize = Cout * 9 * Cin
    plain = torch.full((n, wsize), float("nan"), device="cuda")
    pb.parle_k_conv_backward_weight(desc, dy, x, scratch, plain)
    both = torch.full((n, wsize + Cout), float("nan"), device="cuda")
    assert pb.parle_k_conv_backward_weight_bias(desc, dy, x, scratch, both)
    for a in range(n):
        xp = torch.nn.functional.pad(x[a].double(), (0, 0, 1, 1, 1, 1))
        d = dy[a].double().reshape(-1, Cout)
        ref = torch.stack([d.t() @ xp[:, r:r + H:stride, c:c + W:stride].reshape(-1, Cin) for r in range(3) for c in range(3)], 1).reshape(-1)
        # products of bf16 values are exact in fp32; what is left is the order of up to 40 960 fp32 sums
        bound = 2e-5 * ref.abs().max()
        assert (plain[a] - ref).abs().max() <= bound
        assert (both[a, :wsize] - ref).abs().max() <= bound
        assert ((both[a, wsize:] - d.sum(0)).abs() <= 2e-6 * d.abs().sum(0)).all()


@pytest.mark.parametrize("case", [(1, 2, 28, 28, 64, 64), (1, 64, 7, 7, 64, 64), (1, 2, 15, 12, 32, 96), (1, 3, 8, 8, 64, 64)])
def test_infinities_at_the_edge_reach_no_other_tap(gpu, case):
    """A wavefront multiplies whole rows of 16 or 8 pixels: what an infinite pixel in the last column or row meets beyond the
    image may not turn a finite result into NaN."""
    torch, pb = gpu
    n, B, H, W, Cin, Cout = case
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((n, B, H, W, Cin), generator=gen, device="cuda").bfloat16()
    x[0, 0, H // 2, W - 1, 1] = float("inf")
    x[0, 1, H - 1, W // 2, 2] = float("inf")
    x[0, 1, H - 1, W - 1, 3] = float("inf")
    dy = torch.randn((n, B, H, W, Cout), generator=gen, device="cuda").bfloat16().abs() + 0.5
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, 3, 1, 1)
    scratch = torch.empty(max(pb.parle_k_conv_scratch_bytes(desc), 256), dtype=torch.uint8, device="cuda")
    dw = torch.zeros((n, Cout, 3, 3, Cin), device="cuda")
    pb.parle_k_conv_backward_weight(desc, dy, x, scratch, dw)
    xp = torch.nn.functional.pad(x[0].float(), (0, 0, 1, 1, 1, 1))
    # the taps under which the infinite pixel meets a pixel of dy
    reached = torch.stack([torch.stack([~torch.isfinite(xp[:, r:r + H, c:c + W]).all(dim=2).all(dim=1).all(dim=0)
                                        for c in range(3)]) for r in range(3)])
    assert reached.any() and not reached.all()
    assert (torch.isinf(dw[0]) == reached).all() and not torch.isnan(dw).any()
