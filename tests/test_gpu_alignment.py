"""Tensors that start at an odd element (a view into a larger one) give the same bits as aligned ones, in the kernels that
load and store several elements at a time: the projection's bias in every tile shape of the GEMM, and everything the
kernels for fp32 caches and small or head_dim 64 problems take."""
import pytest
import torch

from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs
from tests.harness import GpuLayerCache

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _at(t, offset):
    """A copy of t on the GPU that starts `offset` elements behind a 16-byte boundary."""
    base = torch.zeros(t.numel() + offset, dtype=t.dtype, device=DEV)
    v = base[offset:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == offset * t.element_size()
    return v


@pytest.mark.parametrize("shape", range(11))
def test_bias_of_the_tiled_projection(shape, knob):
    print("[case] bias, shape", shape, flush=True)
    knob("FC_PROJ_GEMM_SHAPE", shape)
    B, d, Hq, Hkv, A, S = 2, 256, 5, 1, 150, 170  # seven head slots: the last pair of slabs is half empty
    w = inputs.Workload("t", "bf16", B, d, Hq, Hkv, 128, S, A)
    x, W, bias = inputs.hidden_states(w, 1, A).to(DEV), inputs.weights(w, 1).to(DEV), 3 * inputs.bias(w, 1)
    got = []
    for offset in (0, 1, 3):
        g = GpuLayerCache("bf16", B, d, Hq, Hkv, 128, S, max_rows=A)
        q = _at(torch.full((B, Hq, A, 128), float("nan"), dtype=torch.bfloat16), offset)
        fc.fc_qkv_project_scatter(g.handle, 0, x, W, _at(bias, offset), 7, A, None, q)
        torch.cuda.synchronize()
        got.append((q.clone(), g.k_store.clone(), g.v_store.clone()))
        g.close()
    assert bool(torch.isfinite(got[0][0]).all()) and got[0][1].abs().max() > 0
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("dtype,Hq,Hkv,Dh,A,S", [
    ("f32", 4, 2, 64, 9, 300), ("f32", 2, 1, 128, 40, 90), ("bf16", 4, 2, 64, 9, 300), ("bf16", 4, 1, 128, 5, 70),
])
def test_step_of_the_tile_kernels(dtype, Hq, Hkv, Dh, A, S):
    print("[case] step", dtype, Hq, Hkv, Dh, A, S, flush=True)
    B, d = 2, 40
    w = inputs.Workload("t", dtype, B, d, Hq, Hkv, Dh, S, A)
    x, W, bias = inputs.hidden_states(w, 1, A), inputs.weights(w, 1), inputs.bias(w, 1)
    got = []
    for offset in (0, 1, 2, 3):
        g = GpuLayerCache(dtype, B, d, Hq, Hkv, Dh, S, max_rows=A)
        g.write_rows(0, *inputs.kv_fill(w, 1, S), 0)
        q = _at(torch.full((B, Hq, A, Dh), float("nan"), dtype=g.tdt), offset)
        o = _at(torch.full((B, A, Hq * Dh), float("nan"), dtype=g.tdt), offset)
        fc.fc_qkv_project_scatter(g.handle, 0, _at(x, offset), _at(W, offset), _at(bias, offset), S - A, A, None, q)
        fc.fc_active_attention(g.handle, 0, q, A, S, None, o, g.workspace, g.ws_bytes)
        torch.cuda.synchronize()
        got.append((q.clone(), o.clone(), g.k_store.clone(), g.v_store.clone()))
        g.close()
    assert bool(torch.isfinite(got[0][1]).all())
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
