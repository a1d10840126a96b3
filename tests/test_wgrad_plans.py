"""Split counts of the bf16 3x3 weight gradients that keep all nine taps in a wavefront (host code: the scratch query plans as
the launch does)."""
import pytest

from paper_1707_00424_amd import binding as pb


def splits(n, B, H, W, cin, cout, stride=1):
    size = pb.parle_k_conv_scratch_bytes(pb.parle_conv_desc(1, n, B, H, W, cin, cout, 3, stride, 1))
    return max(size // (n * (cout * 9 * cin + cout) * 4), 1)


@pytest.mark.parametrize("case", [(8, 111, 8, 8, 288, 64), (3, 100, 32, 32, 96, 64)])
def test_two_wavefronts_get_two_workgroups_per_compute_unit(case):
    """64 outputs over an odd number of input tiles run in workgroups of two wavefronts: one for each of 256 compute units
    would leave half of the SIMDs without work."""
    n, cin = case[0], case[4]
    assert splits(*case) * (cin // 32) * n > 256
