"""Error of the fp32 convolution kernels against 64 bits, in the 2-norm: they are sums of six products of bf16 parts, and
a product that is missing or takes a wrong part shows here, far below the tolerances of an elementwise comparison."""
import numpy as np
import pytest

import test_gpu_kernels as tk
from test_gpu_nonfinite import shapes, three_products

gpu = tk.gpu

PAIRS = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def bound(terms):
    """2-norm error of a sum of `terms` products: half an ulp of the result's own rounding, and the accumulators' roundings,
    one per 16 products, which add up like a random walk (measured 0.41e-7, 1.3e-7, 2.6e-7 and 1.1e-6 at 64, 864, 2880 and
    32768 terms); twice that, for other shapes."""
    return 2 * (3e-8 + 6e-9 * np.sqrt(terms))


def parts(a):
    out, rest = [], np.asarray(a, np.float32)
    for _ in range(3):
        out.append(tk.to_bf16_grid(rest))
        rest = rest - out[-1]
    return [p.astype(np.float64) for p in out]


@pytest.mark.parametrize("terms", [72, 864, 10240])
def test_a_missing_product_exceeds_the_bound(terms):
    """Without a GPU: the exact sum of the six products is within the bound, that of any five is not."""
    rng = np.random.default_rng(1)
    a, b = rng.standard_normal((200, terms)).astype(np.float32), rng.standard_normal((terms, 200)).astype(np.float32)
    pa, pb = parts(a), parts(b)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    products = {p: pa[p[0]] @ pb[p[1]] for p in PAIRS}
    total = sum(products.values())
    assert np.linalg.norm(total - ref) < 0.1 * bound(terms) * np.linalg.norm(ref)
    for p in PAIRS:
        assert np.linalg.norm(total - products[p] - ref) > bound(terms) * np.linalg.norm(ref), p


CASES = [
    # n, B, H, W, Cin, Cout, k, stride, pad: every instance of the kernels, contractions of 72 to 10240 products
    (1, 4, 16, 16, 8, 32, 3, 1, 1),       # 32 columns
    (1, 2, 32, 32, 96, 96, 3, 1, 1),      # 96
    (1, 16, 16, 16, 64, 128, 3, 1, 1),    # the columns of a wide layer
    (3, 40, 16, 16, 32, 256, 3, 1, 1),    # ... and with the chip full
    (1, 3, 15, 15, 33, 47, 3, 1, 1),      # odd counts: dword loads, results straight from the accumulators
    (1, 3, 14, 14, 50, 70, 3, 1, 1),      # even counts: 8-byte loads
    (8, 20, 32, 32, 36, 64, 3, 2, 1),     # stride 2, which takes 160 workgroups
    (16, 30, 14, 14, 34, 33, 3, 2, 1),    # ... even counts, seven columns, an odd number of outputs
    (16, 30, 15, 13, 35, 36, 3, 2, 1),    # ... odd ones
    (8, 10, 28, 28, 12, 96, 5, 2, 2),     # ... under a 5 x 5 window
    (2, 3, 12, 12, 20, 50, 5, 1, 0),      # input gradient with an image per workgroup, five taps per wavefront
    (1, 3, 7, 9, 6, 13, 3, 1, 1),         # the same, a channel at a time
    (1, 2, 10, 11, 16, 64, 5, 1, 2),
    (1, 2, 9, 9, 16, 24, 7, 1, 3),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_error_against_64_bits(gpu, case):
    torch, pb = gpu
    rng = np.random.default_rng(2)
    operands = [rng.standard_normal(s).astype(np.float32) for s in shapes(case)]
    _, (_, co, k, _, ci), (_, B, Ho, Wo, _) = shapes(case)
    stride, pad = case[7:]
    refs = tk.oracle_conv(operands[0][0], operands[1][0], None, None, False, stride, pad, operands[2][0])
    split = (ci >= 8, stride == 1, ci >= 12)  # the others are fp32 matrix instructions, which round every second product
    for name, got, ref, terms, runs in zip(("forward", "input gradient", "weight gradient"), three_products(torch, pb, case, *operands),
                                           refs, (k * k * ci, k * k * co, B * Ho * Wo), split):
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert not runs or err < bound(terms), f"{name}: {err:.2e}, bound {bound(terms):.2e}"
