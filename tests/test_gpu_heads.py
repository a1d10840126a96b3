"""Classifier heads at the edges of their class blocks (four classes per block, sixteen at most), against the oracle (the
checks of test_gpu_layers)."""
import pytest

import test_gpu_layers as tl

pytestmark = pytest.mark.gpu
gpu = tl.gpu


@pytest.mark.parametrize("C", [1, 3, 4, 5, 8, 9, 12, 13, 15, 16])
@pytest.mark.parametrize("dtype", [0, 1])
def test_heads_at_class_block_edges(gpu, C, dtype):
    tl.test_classifier_head(gpu, 2, 9, 65, C, C & 1, dtype)
    tl.test_pooling_head(gpu, 2, 5, 5, 13, C, dtype)
