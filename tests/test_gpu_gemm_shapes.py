"""GPU parity of the tiled GEMM's 256 x 256 tile (two slabs, two wave groups an interval apart) and of problems
cut into two launches, at the edges: an odd number of slabs, ragged rows, one and few stages, parts of the
hidden dimension."""
import pytest
import torch

from oracle import fc_oracle as orc
from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs
from tests.harness import assert_close
from tests.test_gpu_unmask import _check_lm_head

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _linear(M, K, N, gated, what):
    print("[case]", what, M, K, N, flush=True)
    x, w = inputs.normal(2, "x", (M, K), 1.0, "bf16"), inputs.normal(2, "w", (N, K), 0.05, "bf16")
    aux = inputs.normal(2, "a", (N, K), 0.05, "bf16") if gated else inputs.normal(2, "r", (M, N), 1.0, "bf16")
    xd, wd, ad = x.to(DEV), w.to(DEV), aux.to(DEV)
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    need = fc.fc_linear_workspace_bytes("bf16", M, K, 2 * N if gated else N)
    ws = torch.empty(max(16, need), dtype=torch.uint8, device=DEV)
    if gated:
        fc.fc_ffn_gate_up("bf16", xd, wd, ad, M, K, N, out, ws)
        ref = orc.ffn_gate_up(inputs.as_oracle(x), inputs.as_oracle(w), inputs.as_oracle(aux), "bf16")
    else:
        fc.fc_linear_residual("bf16", xd, wd, ad, M, K, N, out, ws)
        ref = orc.linear_residual(inputs.as_oracle(x), inputs.as_oracle(w), inputs.as_oracle(aux), "bf16")
    torch.cuda.synchronize()
    assert_close(inputs.as_oracle(out), ref, "bf16", what)


@pytest.mark.parametrize("M,K,N,ksplit", [(257, 256, 384, 1), (33, 320, 128, 1), (512, 1024, 256, 3), (300, 1088, 640, 4)])
def test_two_slab_tile(M, K, N, ksplit, knob):
    knob("FC_LIN_WIDE_SHAPE", "3")
    knob("FC_LIN_KSPLIT", str(ksplit))
    _linear(M, K, N, False, "linear, shape 3, %d parts" % ksplit)
    _linear(M, K, N // 2, True, "gated, shape 3")


def test_two_slab_tile_vocabulary(knob):
    knob("FC_LIN_WIDE_SHAPE", "3")
    x, w = inputs.normal(21, "x", (100, 256), 1.0, "bf16"), inputs.normal(21, "w", (640, 256), 0.03, "bf16")
    _check_lm_head("bf16", x, w, "vocabulary, shape 3")


@pytest.mark.parametrize("M,N,gated", [
    (1200, 53 * 128, False),   # the last two slabs in a second launch
    (1800, 36 * 128, False),   # the last eight rows in a second launch
    (512, 296 * 64, True),     # 256 gated slabs in the 256 x 256 tile, 40 in a smaller one
])
def test_problem_cut_into_two_launches(M, N, gated):
    """At the 7B hidden width, where the planner cuts; against plain fp32 products on the GPU."""
    print("[case] cut", M, N, gated, flush=True)
    K, g = 3584, torch.Generator(device=DEV).manual_seed(5)
    x, w, w2 = (torch.empty(s, device=DEV).normal_(0, d, generator=g).bfloat16() for s, d in (((M, K), 1.0), ((N, K), 0.02), ((N, K), 0.02)))
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(max(16, fc.fc_linear_workspace_bytes("bf16", M, K, 2 * N if gated else N)), dtype=torch.uint8, device=DEV)
    ref = x.float() @ w.float().t()
    if gated:
        fc.fc_ffn_gate_up("bf16", x, w, w2, M, K, N, out, ws)
        ref = torch.nn.functional.silu(ref) * (x.float() @ w2.float().t())
    else:
        fc.fc_linear_residual("bf16", x, w, None, M, K, N, out, ws)
    assert_close(inputs.as_oracle(out), inputs.as_oracle(ref), "bf16", "cut")
