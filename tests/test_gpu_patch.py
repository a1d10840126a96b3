"""The stride-1 3x3 and 5x5 bf16 kernel with operands loaded straight into LDS: each of its tile shapes, one tile and several per
workgroup, ragged channel chunks and column blocks, images that end inside a tile, and every form of the epilogue, against
plain products in 64 bits."""
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu

CASES = [
    # n, B, H, W, Cin, Cout: tile shape (pixels x channels, last column block) of the forward pass
    (2, 3, 16, 16, 24, 40),     # 128 x 64, half of the columns padding, one ragged chunk of channels
    (1, 200, 32, 32, 16, 64),   # 128 x 64, 1600 tiles on 768 workgroups
    (1, 100, 28, 28, 40, 96),   # 128 x 96, rows of 28, tiles across images
    (1, 53, 32, 32, 16, 160),   # 128 x 96 and 64
    (1, 256, 32, 32, 40, 64),   # 256 x 64, two tiles each
    (1, 160, 32, 32, 72, 96),   # 256 x 96, 640 tiles on 512 workgroups, three chunks
    (3, 14, 24, 24, 16, 160),   # 256 x 96 and 64
    (1, 64, 32, 32, 32, 128),   # 256 x 128
    (1, 1023, 8, 8, 16, 120),   # same, four images per tile and a shorter ring of weight tiles, ragged everywhere
    (1, 25, 32, 32, 64, 320),   # 256 x 128 and 64
    (1, 100, 32, 32, 16, 320),  # same, both widths several tiles per workgroup
    (1, 399, 8, 8, 32, 304),    # same with four images per tile, the narrow block ragged
    # workgroups that go from one replica to the next under a single chunk of channels: their three tiles lie in three replicas,
    # and the bias of the third goes where that of the first was
    (3, 128, 32, 32, 32, 32),   # 256 x 64
    (5, 43, 32, 32, 16, 64),    # 128 x 64
    # ... and several chunks, the tiles of a replica no multiple of eight
    (7, 33, 27, 29, 40, 64),    # 256 x 64, a ragged last tile in each replica
    (5, 57, 28, 28, 40, 96),    # 256 x 96
    (3, 86, 28, 28, 40, 160),   # 256 x 96 and 64
    (3, 31, 32, 32, 40, 304),   # 256 x 128 and 64
    # contractions long enough that an epilogue with something to read runs on wide tiles
    (1, 256, 32, 32, 96, 96),   # 256 x 96
    (1, 384, 16, 16, 320, 320),  # 256 x 128 and 64, several tiles per workgroup
    (2, 385, 8, 8, 320, 632),   # same, and a shorter ring of weight tiles
]


def _products64(torch, x, w, transpose):
    """``[B, H, W, C]`` with ``[Cout, k, k, Cin]``; transposed: the input gradient."""
    B, H, W, _ = x.shape
    k = w.shape[1]
    xp = torch.nn.functional.pad(x.double(), (0, 0) + (k // 2,) * 4)
    out = 0
    for r in range(k):
        for c in range(k):
            tap = xp[:, r:r + H, c:c + W].reshape(B * H * W, -1)
            m = w[:, k - 1 - r, k - 1 - c] if transpose else w[:, r, c].t()
            out = out + tap @ m.double().contiguous()
    return out.reshape(B, H, W, -1)


@pytest.mark.parametrize("case,k", [(c, 3) for c in CASES] + [
    ((2, 3, 16, 16, 24, 40), 5), ((1, 60, 28, 28, 40, 96), 5), ((1, 140, 32, 32, 16, 64), 5), ((3, 14, 24, 24, 16, 160), 5),
    ((1, 64, 32, 32, 32, 128), 5), ((1, 201, 8, 8, 16, 304), 5), ((1, 65, 7, 7, 72, 64), 5)])
def test_shapes_and_epilogues(gpu, case, k):
    torch, pb = gpu
    n, B, H, W, Cin, Cout = case
    gen = torch.Generator(device="cuda").manual_seed(sum(case))

    def normal(*shape, std=1.0, dtype=torch.bfloat16):
        return (torch.randn(shape, generator=gen, device="cuda") * std).to(dtype)

    x, dy, resid, mask, prev = (normal(n, B, H, W, c) for c in (Cin, Cout, Cout, Cin, Cin))
    w = normal(n, Cout, k, k, Cin, std=(k * k * Cin) ** -0.5)
    bias = normal(n, Cout, dtype=torch.float32)
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, k, 1, k // 2)
    wt = torch.empty_like(w)

    def forward(bias, resid, relu):
        y = torch.full_like(dy, float("nan"))
        pb.parle_k_conv_forward(desc, x, w, bias, resid, relu, y)
        return y

    def backward(mask, onto):
        g = torch.full_like(x, float("nan")) if onto is None else onto.clone()
        pb.parle_k_conv_backward_data(desc, dy, w, mask, int(onto is not None), wt, g)
        return g

    def near(name, got, ref):
        # half a bf16 ulp (2^-9) on the store and room for the order of the sums
        bound = 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().max()
        worst = ((got.double() - ref).abs() - bound).max().item()
        assert worst <= 0, f"{name}: {worst:.3e} outside tolerance"

    for a in range(n):
        y = _products64(torch, x[a], w[a], False)
        g = _products64(torch, dy[a], w[a], True)
        b, r, m = bias[a].double(), resid[a].double(), mask[a] > 0
        near("plain", forward(None, None, 0)[a], y)
        near("bias, ReLU", forward(bias, None, 1)[a], (y + b).relu())
        near("bias, residual", forward(bias, resid, 0)[a], y + b + r)
        near("residual, ReLU", forward(None, resid, 1)[a], (y + r).relu())
        near("gradient", backward(None, None)[a], g)
        near("gradient, mask", backward(mask, None)[a], g * m)
        near("gradient, added", backward(None, prev)[a], g + prev[a].double())
        near("gradient, mask, added", backward(mask, prev)[a], g * m + prev[a].double())


@pytest.mark.parametrize("case", [
    # n, B, H, W, Cin, Cout, k, stride: layers whose whole contraction is one tile, epilogue in registers
    (2, 3, 32, 32, 3, 96, 3, 1),
    (1, 5, 15, 13, 3, 16, 3, 1),     # a ragged last tile, half of the columns padding
    (1, 2, 16, 16, 3, 136, 3, 1),    # two column blocks, the second ragged
    (2, 3, 16, 16, 16, 64, 1, 1),    # whole vectors
    (1, 3, 9, 7, 24, 40, 1, 2),      # same, stride 2, a contraction of three vectors
    (1, 2, 11, 11, 5, 24, 1, 1),     # 1 x 1 gathered value by value
])
def test_small_contractions(gpu, case):
    torch, pb = gpu
    n, B, H, W, Cin, Cout, k, stride = case
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn((n, B, H, W, Cin), generator=gen, device="cuda").bfloat16()
    w = (torch.randn((n, Cout, k, k, Cin), generator=gen, device="cuda") * (k * k * Cin) ** -0.5).bfloat16()
    bias = torch.randn((n, Cout), generator=gen, device="cuda")
    P, Q = (H - 1) // stride + 1, (W - 1) // stride + 1
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, k, stride, k // 2)
    for relu in (0, 1):
        y = torch.full((n, B, P, Q, Cout), float("nan"), dtype=torch.bfloat16, device="cuda")
        pb.parle_k_conv_forward(desc, x, w, bias, None, relu, y)
        for a in range(n):
            xp = torch.nn.functional.pad(x[a].double(), (0, 0) + (k // 2,) * 4)
            ref = bias[a].double() + sum(xp[:, r:r + H:stride, c:c + W:stride].reshape(-1, Cin) @ w[a][:, r, c].double().t().contiguous()
                                         for r in range(k) for c in range(k)).reshape(B, P, Q, Cout)
            ref = ref.relu() if relu else ref
            # half a bf16 ulp on the store and room for the order of the sums
            assert ((y[a].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2e-5 * ref.abs().max()).all()
