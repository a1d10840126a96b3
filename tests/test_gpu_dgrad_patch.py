"""Backward-data of stride-2 3x3 layers with the output-gradient patch in LDS: one tile and several per workgroup, ragged channel
chunks and column blocks, odd image sides, images that end inside a tile, and every form of the epilogue, against plain
products in 64 bits."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

CASES = [
    # n, B, H, W, Cin, Cout
    (1, 1, 32, 32, 32, 32),     # eight workgroups for two tiles, one chunk of channels
    (2, 3, 32, 32, 40, 24),     # the second column block and the only chunk ragged
    (3, 128, 32, 32, 16, 40),   # 768 tiles: one round of three workgroups per compute unit; two chunks, one of 8 channels
    (3, 129, 32, 32, 64, 64),   # 1548 items on 768 workgroups, the next replica's weights behind the last tile of one
    (7, 40, 32, 32, 64, 8),     # several tiles of one ragged chunk each
    (1, 300, 16, 16, 72, 96),   # two images per tile
    (5, 61, 15, 15, 64, 64),    # odd sides: no pixel in the last odd row and column
    (2, 50, 28, 27, 32, 72),    # one of them
    (2, 33, 7, 7, 32, 32),      # images of 4 x 4 positions, seven per tile
    (1, 20, 14, 30, 136, 32),   # rows of 15 positions
    (1, 9, 8, 96, 32, 32),      # rows of 48
    (1, 4, 16, 16, 1024, 32),   # 32 column blocks
]

# bf16 layers of this kind that k_dgrad_s2 keeps: images whose sides are powers of two and output channels in multiples of 32, with
OTHERS = [
    (2, 3, 32, 32, 36, 64),     # input channels in multiples of 4 only
    (1, 5, 16, 16, 100, 32),    # same, the second column block ragged
    (1, 2, 128, 128, 32, 32),   # rows of 64 positions, which fill no tile of 128 with their patch
    (1, 1, 16, 128, 64, 96),
]


def _gradient64(torch, dy, w, H, W):
    """``dy`` [B, P, Q, Cout], ``w`` [Cout, 3, 3, Cin]."""
    B, P, Q, _ = dy.shape
    out = torch.zeros((B, 2 * P + 2, 2 * Q + 2, w.shape[3]), dtype=torch.float64, device=dy.device)
    for r in range(3):
        for c in range(3):
            out[:, r:r + 2 * P:2, c:c + 2 * Q:2] += (dy.double().reshape(B * P * Q, -1) @ w[:, r, c].double().contiguous()).reshape(B, P, Q, -1)
    return out[:, 1:1 + H, 1:1 + W]


@pytest.mark.parametrize("case", CASES + OTHERS)
def test_sizes_and_epilogues(gpu, case):
    torch, pb = gpu
    n, B, H, W, Cin, Cout = case
    P, Q = (H + 1) // 2, (W + 1) // 2
    gen = torch.Generator(device="cuda").manual_seed(sum(case))

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16()

    dy, mask, prev = normal(n, B, P, Q, Cout), normal(n, B, H, W, Cin), normal(n, B, H, W, Cin)
    w = normal(n, Cout, 3, 3, Cin, std=(9 * Cout) ** -0.5)
    wt = torch.empty_like(w)
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, 3, 2, 1)

    def backward(mask, onto):
        g = torch.full_like(prev, float("nan")) if onto is None else onto.clone()
        pb.parle_k_conv_backward_data(desc, dy, w, mask, int(onto is not None), wt, g)
        return g

    def near(name, got, ref):
        # half a bf16 ulp (2^-9) on the store and room for the order of the sums
        bound = 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().max()
        worst = ((got.double() - ref).abs() - bound).max().item()
        assert worst <= 0, f"{name}: {worst:.3e} outside tolerance"

    got = backward(None, None), backward(mask, None), backward(None, prev), backward(mask, prev)
    for a in range(n):
        g, m = _gradient64(torch, dy[a], w[a], H, W), mask[a] > 0
        near("gradient", got[0][a], g)
        near("mask", got[1][a], g * m)
        near("added", got[2][a], g + prev[a].double())
        near("mask, added", got[3][a], g * m + prev[a].double())
