"""Stride-2 3x3 layers loaded straight into LDS, by patches of parity classes and tap by tap: every tile shape of both kernels, one tile
and several per workgroup, ragged channel chunks and column blocks, odd image sides, images that end inside a tile, against plain products in 64
bits and, bit for bit, against the kernels that run these layers with a residual or with column sums; and whole evaluations against
the same network in 64 bits with every stored value rounded."""
import pytest

import test_gpu_eval_norm as te
from paper_1707_00424_amd import synth

pytestmark = pytest.mark.gpu
gpu = te.gpu

CASES = [
    # widths of the two groups, image sides, images: tile shapes (outputs x channels) of the two stride-2 layers; inputs of 33 to 127
    # channels tap by tap
    (64, 128, 32, 32, 3),     # tap by tap; 128 x 64
    (24, 40, 32, 32, 21),     # ragged chunks and column blocks; tap by tap, steps across taps
    (96, 192, 32, 32, 300),   # tap by tap, 128 x 96; 128 x 96, two images per tile
    (160, 32, 32, 32, 300),   # 256 x 64 with several tiles in some workgroups; 128 x 64
    (16, 640, 32, 32, 130),   # 128 x 64; 256 x 64 on small images, four per tile
    (136, 72, 28, 28, 700),   # 256 x 64 on rows of 14, images across tiles
    (32, 160, 15, 15, 70),    # odd sides twice: 8 x 8 and 4 x 4 outputs
    (24, 136, 14, 30, 90),    # rows of 15; outputs of 4 x 8 from 7 x 15
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
    (1, 20, 32, 32, 136, 96),   # 128 x 96, four chunks and a ragged one
    (5, 61, 15, 15, 128, 64),   # odd sides: no odd row and column behind the last even ones
    (1, 33, 28, 27, 136, 96),   # one of them
    (2, 33, 7, 7, 136, 32),     # outputs of 4 x 4, seven images per tile
    (3, 128, 32, 32, 32, 128),  # 256 x 64, 768 workgroups' worth on 512, a single chunk
    (3, 129, 32, 32, 136, 64),  # 256 x 64, the next replica's weights and bias behind the last tile of one
    (3, 129, 16, 16, 128, 640), # 256 x 64, smaller images
    (3, 130, 32, 32, 24, 96),   # 256 x 96, a single ragged chunk
    (1, 600, 28, 28, 136, 96),  # 256 x 96, rows of 14
    (7, 21, 24, 40, 128, 192),  # 256 x 96, two column blocks
    (2, 20, 16, 16, 256, 160),  # 128 x 64, eight chunks
    # tap by tap
    (2, 20, 32, 32, 96, 96),    # 128 x 64, 80 tiles in two column blocks
    (1, 1, 1, 1, 40, 8),        # one output, one tap inside the image
    (3, 2, 2, 3, 48, 24),       # windows wider than the image; ragged everything
    (2, 7, 7, 9, 40, 136),      # steps that span two taps, 8 values in the last one
    (2, 5, 15, 12, 120, 72),    # ... 24 values
    (2, 33, 7, 7, 256, 136),    # channels beyond 127 on a size of no full patches
    (1, 3, 130, 6, 64, 32),     # rows wider and columns narrower than a tile
    (3, 67, 32, 32, 48, 96),    # 128 x 96
    (2, 130, 16, 16, 104, 256), # 128 x 128, two column blocks
    (2, 1001, 15, 15, 40, 64),  # 256 x 64, the last tile of a replica a quarter full
    (3, 131, 32, 32, 40, 136),  # 256 x 96, two column blocks, the second ragged
    (5, 103, 32, 32, 64, 128),  # 256 x 128
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

    def forward(b, relu, resid=None):
        y = torch.full((n, B, P, Q, Cout), float("nan"), dtype=torch.bfloat16, device="cuda")
        pb.parle_k_conv_forward(desc, x, w, b, resid, relu, y)
        return y

    got = forward(None, 0), forward(bias, 1)
    # the order of sums is one: nothing added, as a residual, changes no bit; nor do column sums
    nothing = torch.zeros_like(got[0])
    assert torch.equal(forward(None, 0, nothing), got[0]) and torch.equal(forward(bias, 1, nothing), got[1])
    y = torch.full_like(got[0], float("nan"))
    partial = torch.empty((n * 1024 * 2 * Cout,), dtype=torch.float64, device="cuda")
    pb.parle_k_conv_forward_colsums(desc, x, w, None, y, partial, 1024)
    assert torch.equal(y, got[0])
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
