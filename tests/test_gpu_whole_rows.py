"""GPU parity of the whole-row linear kernels where their ranges end: fewer items than compute units, one item, half
items, and vocabularies that are no multiple of anything."""
import pytest

from paper_2505_21467_amd import inputs
from tests.test_gpu_gemm_shapes import _linear
from tests.test_gpu_unmask import _check_lm_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,gated", [
    (32, 3584, 8, False), (17, 3584, 264, False), (1, 4096, 24, False), (16, 3584, 4, True), (31, 4096, 52, True),
    (32, 512, 4104, False), (5, 512, 2052, True),
])
def test_few_items(M, K, N, gated, knob):
    """By default most of these are streamed through LDS; with a number of workgroups named, in whole rows."""
    _linear(M, K, N, gated, "few outputs")
    knob("FC_LIN_WGS", "256")
    _linear(M, K, N, gated, "whole rows")


@pytest.mark.parametrize("M,K,N,gated", [
    (3, 4096, 8216, False), (18, 3584, 8456, False), (31, 4096, 8448, False),  # more than 8192 outputs
    (2, 4096, 8324, True), (19, 3584, 8324, True), (17, 4096, 8252, True),     # and no whole slabs
])
def test_many_items(M, K, N, gated):
    _linear(M, K, N, gated, "whole rows")


@pytest.mark.parametrize("M,K,V", [
    (20, 3584, 1001), (32, 512, 15999), (1, 4096, 9), (16, 512, 8193),            # up to 16384 entries: streamed through LDS
    (3, 512, 17239), (2, 4096, 16418), (17, 4096, 16461), (9, 3584, 16386), (32, 3584, 16391),  # more: whole rows at hidden 3584 and 4096
])
def test_odd_vocabulary(M, K, V):
    print("[case] odd vocabulary", M, K, V, flush=True)
    x, w = inputs.normal(31, "x", (M, K), 1.0, "bf16"), inputs.normal(31, "w", (V, K), 0.03, "bf16")
    _check_lm_head("bf16", x, w, "vocabulary of %d" % V)
