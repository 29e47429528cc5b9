"""The non-temporal hint changes where bytes wait and nothing else: a layer of a model whose weights and cache exceed the
memory-side cache gives the bits that the same layer gives by itself, in every kernel that has the hint (runs of pairs and of
outputs, tiles of the tiled GEMM with one tile of rows, split-KV attention)."""
import pytest
import torch

from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,d,Hq,Hkv,F,A,L", [
    (1, 2048, 16, 4, 4096, 3, 40),      # runs of pairs and outputs, 16 rows
    (1, 2048, 16, 4, 6144, 32, 300),    # 32 rows, ragged runs
    (2, 2048, 16, 4, 18944, 24, 90),    # 48 rows: gated in 64-row tiles
    (1, 3584, 4, 4, 8192, 17, 2500),    # attention in ranges of keys, one workgroup each; hidden dimension of W_2 in parts
    (4, 1024, 24, 24, 10240, 32, 3000),  # 128-row tiles
    (3, 4096, 40, 8, 4096, 33, 1000),  # 99 rows, rotated starts
    (8, 2048, 16, 4, 18944, 32, 90),   # 256 rows: tiles of 256, gated by dealt pairs
    (5, 3584, 28, 4, 8192, 33, 60),    # 165 rows
    (1, 4096, 32, 8, 6144, 200, 70),   # 200 rows of one sequence
])
def test_hint_keeps_the_bits(B, d, Hq, Hkv, F, A, L):
    print("[case] read once", B, d, Hq, Hkv, F, A, L, flush=True)
    Dh, S, E = 128, L + A, Hq * 128
    gen = torch.Generator(device=DEV).manual_seed(A)

    def rnd(shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(mean, std, generator=gen)

    t = {"norm1": rnd((d,), 0.1, 1.0), "w_qkv": rnd(((Hq + 2 * Hkv) * Dh, d), 0.02), "b_qkv": rnd(((Hq + 2 * Hkv) * Dh,), 0.02),
         "w_out": rnd((d, E), 0.02), "norm2": rnd((d,), 0.1, 1.0), "w_gate": rnd((F, d), 0.02), "w_up": rnd((F, d), 0.02),
         "w_down": rnd((d, F), 0.02)}
    wt = fc.make_layer_weights(d_ff=F, eps=1e-6, **t)
    x, k, v = rnd((B, A, d)), rnd((B, Hkv, L, Dh)), rnd((B, Hkv, L, Dh))
    layer_bytes = 2 * sum(t[n].numel() for n in ("w_qkv", "w_out", "w_gate", "w_up", "w_down")) + 4 * B * Hkv * S * Dh
    many = (256 << 20) // layer_bytes + 1
    assert many > 1  # (alone: within the memory-side cache)
    got = []
    for layers in (1, many):
        cfg = fc.make_config(layers, B, d, Hq, Hkv, Dh, S, "bf16")
        handle = fc.fc_cache_alloc(cfg)
        fc.fc_cache_write_rows(handle, 0, k, v, 0, L)
        y = torch.full_like(x, float("nan"))
        ws = torch.empty(fc.fc_full_layer_workspace_bytes(cfg, F, A), dtype=torch.uint8, device=DEV)
        fc.fc_full_layer_step(handle, 0, wt, x, L, A, None, S, y, ws)
        kk, vv = torch.empty((B, Hkv, S, Dh), dtype=torch.bfloat16, device=DEV), torch.empty((B, Hkv, S, Dh), dtype=torch.bfloat16, device=DEV)
        fc.fc_cache_read_rows(handle, 0, kk, vv, 0, S)
        torch.cuda.synchronize()
        fc.fc_cache_free(handle)
        got.append((y, kk, vv))
    assert torch.isfinite(got[0][0].float()).all()
    for a, b in zip(*got):
        assert torch.equal(a, b)
