"""Stride-2 3x3 layers that run as four stride-1 convolutions of parity classes: every tile shape of that kernel, one
tile and several per workgroup, ragged channel chunks and column blocks, odd image sides, images that end inside a tile, against
plain products in 64 bits, and whole evaluations against the same network in 64 bits with every stored value rounded."""
import pytest

import test_gpu_eval_norm as te
from paper_1707_00424_amd import synth

pytestmark = pytest.mark.gpu
gpu = te.gpu

CASES = [
    # widths of the two groups, image sides, images: tile shapes (outputs x channels) of the two stride-2 layers
    (64, 128, 32, 32, 3),     # 128 x 64 twice
    (24, 40, 32, 32, 21),     # same, ragged chunks and column blocks
    (96, 192, 32, 32, 300),   # 256 x 96, two tiles in some workgroups; 128 x 96, two images per tile
    (64, 32, 32, 32, 1100),   # 256 x 64, three tiles per workgroup; 128 x 64
    (16, 640, 32, 32, 130),   # 256 x 64 on small images, four per tile: a shorter ring of weight tiles
    (96, 72, 28, 28, 700),    # 256 x 96 on rows of 14, images across tiles; 128 x 64 on rows of 7
    (32, 96, 15, 15, 70),     # odd sides twice: 8 x 8 and 4 x 4 outputs
    (48, 56, 14, 30, 90),     # rows of 15; outputs of 4 x 8 from 7 x 15
]


@pytest.mark.parametrize("case", CASES)
def test_evaluations(gpu, case):
    torch, pb = gpu
    ca, cb, H, W, count = case
    cfg = pb.make_config(model=pb.MODEL_ALLCNN_C, n_replicas=1, batch=count, compute_bf16=1, in_h=H, in_w=W, in_c=3, n_classes=10,
                         arch=(ca, cb, 0, 0), eta_inner=0.01, eta_outer=0.01, gamma0=0.03, rho0=1.0)
    layout = pb.parle_query_layout(cfg)
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    row = torch.as_tensor(synth.init_params(layout, 5, "he_normal")).cuda()
    for s in layout:
        if s["kind"] == "bias":
            row[s["offset"]:s["offset"] + s["size"]] = 0.1 * torch.randn(s["size"], generator=gen, device="cuda")
    P = pb.Parle(cfg, row[None].contiguous())
    images = torch.randn((count, H, W, 3), generator=gen, device="cuda")
    labels = torch.randint(0, 10, (count,), generator=gen, device="cuda", dtype=torch.int32)

    bf = lambda t: t.bfloat16().double()  # noqa: E731
    seg = {s["name"]: row[s["offset"]:s["offset"] + s["size"]].reshape(s["shape"]).double() for s in layout}
    logits = []
    for part in bf(images).split(64):
        x = part
        for i, stride in enumerate((1, 1, 2, 1, 1, 2, 1, 1, 1)):
            w = seg[f"conv{i + 1}.w"]
            w = w if w.dim() == 4 else w.reshape(w.shape[0], 1, 1, w.shape[1])
            x = te._conv(torch, x, bf(w), stride) + seg[f"conv{i + 1}.b"]
            x = bf(x.relu() if i < 8 else x)
        logits.append(x.mean((1, 2)))
    each = torch.nn.functional.cross_entropy(torch.cat(logits), labels.long(), reduction="none")
    # every image by its place: parts of the set, each in a call of its own, and the whole
    for a, b in ((0, count), (0, 1), (count // 3, count // 3 + 2), (count // 2, count)):
        b = min(b, count)
        loss, _, _ = P.parle_eval(0, images[a:b].clone(), labels[a:b].clone())
        ref = each[a:b].mean().item()
        # stored values land on the other side of a rounding in a few of 10^5 cases: 2^-9 of one value among thousands
        assert abs(loss - ref) <= 2e-3 * abs(ref), (a, b, loss, ref)


LAYERS = [
    # n, B, H, W, Cin, Cout: tile shape (outputs x channels)
    (1, 1, 32, 32, 32, 32),     # 128 x 64, two tiles, a single chunk
    (2, 3, 32, 32, 24, 40),     # ragged everywhere
    (1, 20, 32, 32, 40, 96),    # 128 x 96
    (5, 61, 15, 15, 64, 64),    # odd sides: no odd row and column behind the last even ones
    (1, 33, 28, 27, 32, 96),    # one of them
    (2, 33, 7, 7, 40, 32),      # outputs of 4 x 4, seven images per tile
    (3, 128, 32, 32, 32, 128),  # 256 x 64, 768 workgroups' worth on 512, a single chunk
    (3, 129, 32, 32, 72, 64),   # 256 x 64, the next replica's weights and bias behind the last tile of one
    (3, 129, 16, 16, 64, 640),  # 256 x 64, smaller images: a shorter ring of weight tiles
    (3, 130, 32, 32, 40, 96),   # 256 x 96
    (1, 600, 28, 28, 64, 96),   # 256 x 96, rows of 14
    (7, 21, 24, 40, 16, 192),   # 256 x 96, two column blocks
]


@pytest.mark.parametrize("case", LAYERS)
def test_layers(gpu, case):
    torch, pb = gpu
    n, B, H, W, Cin, Cout = case
    P, Q = (H + 1) // 2, (W + 1) // 2
    gen = torch.Generator(device="cuda").manual_seed(sum(case))
    x = torch.randn((n, B, H, W, Cin), generator=gen, device="cuda").bfloat16()
    w = (torch.randn((n, Cout, 3, 3, Cin), generator=gen, device="cuda") * (9 * Cin) ** -0.5).bfloat16()
    bias = torch.randn((n, Cout), generator=gen, device="cuda")
    desc = pb.parle_conv_desc(1, n, B, H, W, Cin, Cout, 3, 2, 1)
    got = []
    for b, relu in ((None, 0), (bias, 1)):
        y = torch.full((n, B, P, Q, Cout), float("nan"), dtype=torch.bfloat16, device="cuda")
        pb.parle_k_conv_forward(desc, x, w, b, None, relu, y)
        got.append(y)
    # with column sums: the same values, and their sums and those of their squares over all rows
    cap = 1024
    y = torch.full_like(got[0], float("nan"))
    partial = torch.full((n * cap * 2 * Cout,), float("nan"), dtype=torch.float64, device="cuda")
    S = pb.parle_k_conv_forward_colsums(desc, x, w, None, y, partial, cap)
    assert torch.equal(y, got[0])
    if S:
        sums = partial[:n * S * 2 * Cout].reshape(n, S, 2, Cout).sum(1)
        v = y.double().reshape(n, -1, Cout)
        # fp32 sums of 256 values each
        assert ((sums[:, 0] - v.sum(1)).abs() <= 1e-5 * v.abs().sum(1)).all()
        assert ((sums[:, 1] - (v * v).sum(1)).abs() <= 1e-5 * (v * v).sum(1)).all()
        assert partial[n * S * 2 * Cout:].isnan().all()
    for a in range(n):
        xp = torch.nn.functional.pad(x[a].double(), (0, 0, 1, 2, 1, 2))
        ref = 0
        for r in range(3):
            for c in range(3):
                ref = ref + xp[:, r:r + 2 * P:2, c:c + 2 * Q:2].reshape(B * P * Q, Cin) @ w[a][:, r, c].double().t().contiguous()
        ref = ref.reshape(B, P, Q, Cout)
        for y, want in ((got[0], ref), (got[1], (ref + bias[a].double()).relu())):
            # half a bf16 ulp (2^-9) on the store and room for the order of the sums
            worst = ((y[a].double() - want).abs() - 2.0 ** -8 * want.abs() - 2e-5 * want.abs().max()).max().item()
            assert worst <= 0, f"{worst:.3e} outside tolerance"
