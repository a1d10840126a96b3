"""Operands at and beyond the ends of the number format, through the convolution kernels: infinities and NaN reach the
results they reach in plain arithmetic and no others."""
import numpy as np
import pytest

import test_gpu_kernels as tk

pytestmark = pytest.mark.gpu
gpu = tk.gpu


def shapes(case):
    n, B, H, W, Cin, Cout, k, stride, pad = case
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    return (n, B, H, W, Cin), (n, Cout, k, k, Cin), (n, B, Ho, Wo, Cout)


def weight_and_bias_gradient(torch, pb, case, dtype, x, dy):
    """Replica 0's weight gradient, and its bias gradient where the kernel takes it along (else None)."""
    _, ws, _ = shapes(case)
    desc = pb.parle_conv_desc(dtype, *case)
    dx_, ddy = tk.upload(torch, x, dtype), tk.upload(torch, dy, dtype)
    wsize, cout = int(np.prod(ws[1:])), ws[1]
    scratch = torch.zeros(max(pb.parle_k_conv_scratch_bytes(desc) // 4, 4), dtype=torch.float32, device="cuda")
    gw = torch.zeros((ws[0], wsize + cout), dtype=torch.float32, device="cuda")
    took = pb.parle_k_conv_backward_weight_bias(desc, ddy, dx_, scratch, gw)
    torch.cuda.synchronize()
    gw = tk.download(gw[0])
    return gw[:wsize].reshape(ws[1:]), (gw[wsize:] if took else None)


def assert_same_kind(name, got, ref):
    """Finite where the reference is and near it, the same infinities, NaN where it has them."""
    fin = np.isfinite(ref)
    assert (np.isfinite(got) == fin).all(), f"{name}: {np.sum(np.isfinite(got) != fin)} of {ref.size} differ in kind"
    inf = np.isinf(ref)
    assert (got[inf] == ref[inf]).all(), name
    assert np.isnan(got[np.isnan(ref)]).all(), name
    if fin.any():
        tk.assert_near(name, got[fin], ref[fin], 1e-6, 2e-5 * np.abs(ref[fin]).max())


RAGGED = [
    # dtype, (n, B, H, W, Cin, Cout, k, stride, pad): output rows that are no multiple of eight columns
    (0, (1, 3, 7, 7, 24, 36, 3, 1, 1)),
    (0, (1, 2, 12, 12, 20, 50, 5, 1, 2)),    # four dead columns under a 5 x 5 window
    (0, (1, 2, 9, 28, 16, 32, 3, 1, 1)),
    (0, (1, 2, 9, 28, 16, 32, 3, 2, 1)),     # stride 2: even and odd columns
    (0, (1, 2, 16, 15, 13, 40, 7, 1, 3)),    # three groups of taps per window row
    (1, (1, 3, 7, 7, 20, 36, 3, 1, 1)),      # bf16, two channels per lane
    (1, (1, 2, 9, 28, 17, 33, 3, 1, 1)),     # one channel per lane
    (1, (1, 2, 9, 28, 18, 34, 3, 2, 1)),
    (1, (1, 2, 9, 11, 18, 34, 5, 1, 0)),     # two groups of taps, whose values beyond the row are pixels of the image
    (0, (1, 2, 9, 11, 18, 34, 7, 1, 0)),
]


@pytest.mark.parametrize("dtype,case", RAGGED)
def test_infinity_in_the_last_column_stays_in_its_taps(gpu, dtype, case):
    """The last column of x reaches the taps that some output column reads it through, and no tap beyond the row."""
    torch, pb = gpu
    stride, pad = case[7:]
    xs, ws, ys = shapes(case)
    rng = np.random.default_rng(3)
    q = tk.to_bf16_grid if dtype else (lambda a: np.asarray(a, np.float32))
    x, dy = q(rng.standard_normal(xs)), q(rng.standard_normal(ys))
    x[0, 0, 3, -1, 1], x[0, 1, 4, -1, 2], x[0, 1, 5, -2, 12] = np.inf, np.nan, -np.inf
    with np.errstate(invalid="ignore"):
        _, _, ref = tk.oracle_conv(x[0], np.zeros(ws[1:]), None, None, False, stride, pad, dy[0])
    assert np.isfinite(ref[..., 1]).any(), "the case has a tap that the infinity does not reach"
    got, _ = weight_and_bias_gradient(torch, pb, case, dtype, x, dy)
    assert_same_kind("weight gradient", got, ref)


@pytest.mark.parametrize("case", [(1, 3, 7, 7, 24, 36, 3, 1, 1), (1, 2, 16, 16, 16, 32, 3, 1, 1)])
def test_infinite_gradient_leaves_an_infinite_bias_gradient(gpu, case):
    torch, pb = gpu
    xs, ws, ys = shapes(case)
    rng = np.random.default_rng(4)
    x, dy = (rng.standard_normal(s).astype(np.float32) for s in (xs, ys))
    dy[0, 0, 2, 3, 5], dy[0, 1, 1, 1, 6], dy[0, 1, 2, 2, 7] = np.inf, -np.inf, np.nan
    got, bias = weight_and_bias_gradient(torch, pb, case, 0, x, dy)
    assert bias is not None
    with np.errstate(invalid="ignore"):
        ref = dy[0].astype(np.float64).sum(axis=(0, 1, 2))
        _, _, rdw = tk.oracle_conv(x[0], np.zeros(ws[1:]), None, None, False, *case[7:], dy[0])
    assert_same_kind("bias gradient", bias, ref)
    assert_same_kind("weight gradient", got, rdw)


SPLIT = [
    # n, B, H, W, Cin, Cout, k, stride, pad: every form of the kernels that split fp32 values into bf16 parts
    (1, 3, 16, 16, 32, 64, 3, 1, 1),     # results in whole rows
    (1, 3, 15, 15, 33, 47, 3, 1, 1),     # odd counts, results straight from the accumulators
    (16, 24, 14, 14, 50, 20, 3, 2, 1),   # stride 2, which takes 160 workgroups
    (1, 2, 12, 12, 20, 50, 5, 1, 0),     # input gradient with an image per workgroup
    (1, 2, 7, 7, 28, 48, 3, 1, 1),
    (1, 2, 7, 7, 30, 48, 3, 1, 1),       # ... two channels at a time
    (1, 2, 7, 7, 27, 48, 3, 1, 1),       # ... one
]


def three_products(torch, pb, case, x, w, dy):
    """Replica 0's forward result, input gradient and weight gradient in fp32."""
    xs, ws, ys = shapes(case)
    desc = pb.parle_conv_desc(0, *case)
    dx_, dw_, ddy = (tk.upload(torch, a, 0) for a in (x, w, dy))
    y, gx, gw = (torch.zeros(s, dtype=torch.float32, device="cuda") for s in (ys, xs, ws))
    scratch = torch.zeros(max(pb.parle_k_conv_scratch_bytes(desc) // 4, 4), dtype=torch.float32, device="cuda")
    pb.parle_k_conv_forward(desc, dx_, dw_, None, None, 0, y)
    pb.parle_k_conv_backward_data(desc, ddy, dw_, None, 0, torch.zeros_like(dw_), gx)
    pb.parle_k_conv_backward_weight(desc, ddy, dx_, scratch, gw)
    torch.cuda.synchronize()
    return [tk.download(t[0]) for t in (y, gx, gw)]


def assert_within_fp32(case, got, x, w, dy):
    """Every result within the bound of a plain fp32 sum: a rounding of 2^-24 per product, of the sum of their magnitudes."""
    stride, pad = case[7:]
    refs = tk.oracle_conv(x[0], w[0], None, None, False, stride, pad, dy[0])
    sizes = tk.oracle_conv(np.abs(x[0]), np.abs(w[0]), None, None, False, stride, pad, np.abs(dy[0]))
    _, (_, co, k, _, ci), (_, B, Ho, Wo, _) = shapes(case)
    for name, g, ref, size, terms in zip(("forward", "input gradient", "weight gradient"), got, refs, sizes,
                                         (k * k * ci, k * k * co, B * Ho * Wo)):
        outside = ~(np.abs(g - ref) <= terms * 2.0 ** -24 * size)  # NaN counts
        assert not outside.any(), f"{name}: {outside.sum()} of {ref.size} outside"


@pytest.mark.parametrize("case", SPLIT)
def test_operands_beyond_the_largest_bf16_value(gpu, case):
    """Floats from 3.396e38 up round to an infinite bf16 value; their products with small numbers are finite."""
    torch, pb = gpu
    xs, ws, ys = shapes(case)
    big = np.finfo(np.float32).max
    places = [((0, 0, 3, 4, 1), (0, 1, 5, 2, 3)), ((0, 2, 1, 1, 4), (0, 5, 0, 1, 2)), ((0, 0, 2, 2, 5), (0, 1, 1, 3, 0))]
    for turn in range(3):  # x, w, dy in turn
        rng = np.random.default_rng(6)
        operands = [1e-3 * rng.standard_normal(s).astype(np.float32) for s in (xs, ws, ys)]
        first, second = places[turn]
        operands[turn][first], operands[turn][second] = big, -np.float32(3.3962e38)
        assert_within_fp32(case, three_products(torch, pb, case, *operands), *operands)


@pytest.mark.parametrize("scale", [1e-33, 3e-36, 2e-37])
@pytest.mark.parametrize("case", SPLIT)
def test_small_operands_keep_their_bits(gpu, case, scale):
    """Operands whose third bf16 part would be a denormal, down to the end of the normal range: the results are as close as
    plain fp32 sums (2e-7 in 2-norm on such operands; 9e-6 and 1.4e-4 at the two smaller scales with the parts alone)."""
    torch, pb = gpu
    stride, pad = case[7:]
    for turn in range(3):
        rng = np.random.default_rng(8)
        operands = [rng.standard_normal(s).astype(np.float32) for s in shapes(case)]
        operands[turn] *= np.float32(scale)
        refs = tk.oracle_conv(operands[0][0], operands[1][0], None, None, False, stride, pad, operands[2][0])
        names = ("forward", "input gradient", "weight gradient")
        for i, (name, got, ref) in enumerate(zip(names, three_products(torch, pb, case, *operands), refs)):
            err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
            assert err < 1e-6, f"{name}, operand {turn} small: {err:.1e}"


BF16 = [
    # bf16 layers with patches loaded straight into LDS; input gradients read the weights as they lie
    (2, 3, 16, 16, 32, 64, 3, 2, 1),     # stride 2: parity classes in both directions, one chunk forward
    (1, 3, 15, 14, 136, 40, 3, 2, 1),    # ragged chunks, an odd side
    (1, 2, 28, 28, 128, 96, 3, 2, 1),    # rows of 14
    (1, 3, 15, 14, 40, 24, 3, 2, 1),     # forward tap by tap, a last step of 8 values
    (2, 3, 16, 16, 32, 64, 3, 1, 1),
    (1, 4, 9, 14, 40, 72, 3, 1, 1),      # images that end inside a tile
    (1, 3, 16, 16, 32, 96, 5, 1, 2),
]


@pytest.mark.parametrize("case", BF16)
def test_infinities_reach_the_pixels_that_a_window_covers(gpu, case):
    torch, pb = gpu
    stride, pad = case[7:]
    xs, ws, ys = shapes(case)
    rng = np.random.default_rng(9)
    x, w, dy = (tk.to_bf16_grid(rng.standard_normal(s)) for s in (xs, ws, ys))
    w /= 16
    for a in (x, dy):  # corners of the first and last image, an odd and an even place between
        a[0, 0, 0, 0, 1], a[0, 0, -1, -1, 2], a[0, -1, 3, 4, 5], a[0, -1, -1, 0, 7] = np.inf, -np.inf, np.nan, np.inf
    with np.errstate(invalid="ignore"):
        ref, rdx, _ = tk.oracle_conv(x[0], w[0], None, None, False, stride, pad, dy[0])
    desc = pb.parle_conv_desc(1, *case)
    dx_, dw_, ddy = (tk.upload(torch, a, 1) for a in (x, w, dy))
    y, gx = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in (ys, xs))
    pb.parle_k_conv_forward(desc, dx_, dw_, None, None, 0, y)
    pb.parle_k_conv_backward_data(desc, ddy, dw_, None, 0, torch.zeros_like(dw_), gx)
    for name, got, want in (("forward", tk.download(y[0]), ref), ("input gradient", tk.download(gx[0]), rdx)):
        fin = np.isfinite(want)
        assert fin.any() and not fin.all() and (np.isfinite(got) == fin).all(), f"{name}: {np.sum(np.isfinite(got) != fin)} differ in kind"
        inf = np.isinf(want)
        assert (got[inf] == want[inf]).all() and np.isnan(got[np.isnan(want)]).all(), name
        tk.assert_near(name, got[fin], want[fin], *tk.tolerances(1, want[fin]))


@pytest.mark.parametrize("side,place,taps", [(28, (0, 0), [0]), (28, (27, 27), [24]), (17, (0, 3), [0, 1, 2, 3]), (28, (27, 1), [20, 21])])
def test_nan_in_an_image_of_a_first_layer_with_its_pool(gpu, side, place, taps):
    """A ReLU makes zeros of the outputs that a NaN reaches; the weight gradient has NaN at the taps that read it (0 * NaN) and nowhere
    else."""
    torch, pb = gpu
    from paper_1707_00424_amd import synth
    cfg = pb.make_config(model=pb.MODEL_LENET, n_replicas=2, batch=9, in_h=side, in_w=side, in_c=1, n_classes=10, arch=(16, 12, 5 if side > 17 else 4, 24),
                         eta_inner=0.05, eta_outer=0.1, gamma0=0.3, rho0=1.0)
    layout = pb.parle_query_layout(cfg)
    P = pb.Parle(cfg, np.stack([synth.init_params(layout, 3 + a, "uniform") for a in range(2)]))
    gen = torch.Generator(device="cuda").manual_seed(1)
    images = torch.randn((2, 9, side, side, 1), generator=gen, device="cuda")
    images[0, 4, place[0], place[1], 0] = float("nan")
    labels = torch.randint(0, 10, (2, 9), generator=gen, device="cuda").int()
    loss = torch.zeros(2, device="cuda")
    P.parle_inner_step(images, labels, loss)
    assert loss.isfinite().all()
    seg = {s["name"]: P.grad[:, s["offset"]:s["offset"] + s["size"]] for s in layout}
    nan = seg["conv1.w"].reshape(2, 16, -1).isnan()
    want = torch.zeros_like(nan)
    want[0, :, taps] = True
    assert torch.equal(nan, want)
    assert all(g.isfinite().all() for name, g in seg.items() if name != "conv1.w")
