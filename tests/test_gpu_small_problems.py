"""GPU parity of small bf16 problems, which run in the tile kernel up to a number of products: on both sides of the line."""
import numpy as np
import pytest

from paper_2505_21467_amd import inputs
from tests.harness import assert_close
from tests.test_gpu_gemm_shapes import _linear
from tests.test_gpu_parity import _compare_cache, _pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,gated", [
    (8, 1024, 512, False), (32, 2048, 1024, True), (33, 768, 384, False), (74, 512, 520, False), (160, 512, 512, True),
    (75, 1024, 1024, True), (74, 1024, 1024, False), (300, 1024, 1024, False),
    (4, 2048, 2048, False), (12, 6144, 256, False), (33, 4096, 128, False),  # long chains: the tile kernel only for the first
])
def test_small_linear_layers(M, K, N, gated):
    _linear(M, K, N, gated, "small")


@pytest.mark.parametrize("B,d,Hq,Hkv,A", [
    (1, 1024, 4, 1, 20), (2, 512, 4, 2, 37), (1, 384, 4, 2, 20), (1, 384, 3, 1, 74), (2, 512, 8, 2, 100), (1, 256, 4, 4, 60),
    (1, 3072, 2, 1, 9), (1, 5120, 2, 1, 9), (1, 384, 4, 2, 16),  # tile kernel, head-split, neither
])
def test_small_projections(B, d, Hq, Hkv, A):
    print("[case] small projection", B, d, Hq, Hkv, A, flush=True)
    dtype, Dh, L = "bf16", 128, 33
    w, S = inputs.Workload("t", dtype, B, d, Hq, Hkv, Dh, L, A), L + A
    g, o = _pair(dtype, B, d, Hq, Hkv, Dh, S + 5, max_rows=A, fill=0.25)
    K, V = inputs.kv_fill(w, 29, L)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    W, b, X = inputs.weights(w, 29), inputs.bias(w, 29), inputs.hidden_states(w, 29, A)
    Qg, Og = g.step(0, X, W, b, L, S)
    Qo, Oo = o.step(X, W, b, L, S)
    assert_close(Qg, Qo, dtype, "Q")
    assert_close(Og, Oo, dtype, "O")
    written = np.zeros((B, S + 5), bool)
    written[:, L:S] = True
    _compare_cache(g, o, dtype, written=written, what="small projection")
    g.close()
