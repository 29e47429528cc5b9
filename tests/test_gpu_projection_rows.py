"""GPU parity of the projection kernels at the edges of their ranges, with bias and with padded and out-of-range
positions: runs of pairs streamed through LDS (one and two pair tiles, each number of 16-row tiles, ragged last tiles), head-split
beyond hidden 8192 at 33 .. 128 rows, and the sizes where the tiled GEMM and the tile kernel take over."""
import numpy as np
import pytest
import torch

from paper_2505_21467_amd import inputs
from tests.harness import assert_close
from tests.test_gpu_parity import _compare_cache, _pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,d,Hq,Hkv,A", [
    (1, 3584, 4, 1, 33), (1, 3584, 2, 1, 48), (3, 3584, 4, 2, 19), (1, 4096, 3, 1, 65), (4, 3584, 2, 2, 24),
    (2, 4096, 2, 1, 50), (1, 3584, 2, 1, 127), (1, 3584, 2, 1, 128),  # streamed, two to eight tiles of rows
    (1, 3584, 2, 1, 129), (1, 768, 4, 2, 33), (1, 1024, 2, 1, 20),    # more rows; few rows of a small matrix (tile kernel)
    (1, 512, 4, 2, 5), (2, 512, 30, 5, 16), (1, 512, 60, 4, 17),       # hidden 512: runs of few pairs
    (1, 3584, 28, 4, 32), (2, 3584, 30, 5, 8), (1, 3584, 3, 1, 9),     # hidden 3584: runs of 9 or 10 pairs; of few
    (1, 4096, 33, 3, 18), (3, 4096, 1, 1, 5),                          # hidden 4096: runs of 9 or 10 pairs; of few
    (1, 512, 56, 8, 9), (1, 512, 28, 4, 34), (3, 512, 16, 8, 34), (4, 512, 16, 16, 29),  # 16 rows x two pair tiles; 48 rows; 64 rows x one, two
    (1, 10240, 1, 1, 45), (3, 10240, 1, 1, 17), (1, 11264, 1, 1, 74), (1, 10240, 1, 1, 94), (1, 10240, 7, 1, 112),
    (1, 12288, 8, 1, 123),                                             # head-split, three to eight tiles
    (3, 2048, 56, 8, 22), (2, 2048, 112, 16, 35), (1, 1024, 128, 16, 3), (4, 64, 64, 16, 82),  # tiled GEMM: half heads, 48 pairs, 64 rows; 80 pairs
])
def test_projection_rows(B, d, Hq, Hkv, A):
    print("[case] projection rows", B, d, Hq, Hkv, A, flush=True)
    dtype, Dh, L = "bf16", 128, 70
    w, S = inputs.Workload("t", dtype, B, d, Hq, Hkv, Dh, L, A), L + A
    g, o = _pair(dtype, B, d, Hq, Hkv, Dh, S + 7, max_rows=A, fill=0.75)
    K, V = inputs.kv_fill(w, 23, L)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    W, b, X = inputs.weights(w, 23), inputs.bias(w, 23), inputs.hidden_states(w, 23, A)
    gen = torch.Generator().manual_seed(A)
    pos = torch.stack([torch.randperm(S + 7, generator=gen)[:A] for _ in range(B)]).to(torch.int32)
    pos[:, 0] = -1
    pos_o = pos.clone()
    pos[:, 2], pos_o[:, 2] = S + 100, -1
    Qg, Og = g.step(0, X, W, b, 0, S + 7, pos=pos)
    Qo, Oo = o.step(X, W, b, 0, S + 7, pos=pos_o)
    assert_close(Qg, Qo, dtype, "Q")
    assert_close(Og, Oo, dtype, "O")
    written = np.zeros((B, S + 7), bool)
    for bb in range(B):
        written[bb, [int(p) for p in pos_o[bb] if 0 <= int(p) < S + 7]] = True
    _compare_cache(g, o, dtype, written=written, what="projection rows")
    g.close()
