"""The non-temporal hint changes where bytes wait and nothing else: a layer of a model whose weights and cache exceed the
memory-side cache gives the bits that the same layer gives by itself, in every kernel that has the hint (runs of pairs and of
outputs, every tile shape of the tiled GEMM with one tile of rows, split-KV attention; runs of vocabulary entries: see
test_gpu_large_vocabulary.py)."""
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


ROWS = {0: 200, 3: 200, 4: 200, 1: 100, 2: 100, 5: 100, 8: 100, 6: 50, 7: 50, 9: 50, 10: 50}  # tile shape of the tiled GEMM: one tile of rows


@pytest.mark.parametrize("K", [1088, 1024, 2048])  # hidden in stages of 64 and of 128; rotated starts
@pytest.mark.parametrize("shape", sorted(ROWS))
def test_projection_in_every_tile_shape(shape, K, knob):
    print("[case] read once, projection, shape", shape, K, flush=True)
    knob("FC_PROJ_GEMM_SHAPE", str(shape))
    A, Hq, Hkv, Dh = ROWS[shape], 4, 1, 128
    gen = torch.Generator(device=DEV).manual_seed(shape)
    w = torch.empty(((Hq + 2 * Hkv) * Dh, K), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    bias = torch.empty((w.shape[0],), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    x = torch.empty((1, A, K), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    got = []
    for layers in (1, (256 << 20) // (2 * w.numel() + 4 * Hkv * A * Dh) + 1):
        handle = fc.fc_cache_alloc(fc.make_config(layers, 1, K, Hq, Hkv, Dh, A, "bf16"))
        q = torch.full((1, Hq, A, Dh), float("nan"), dtype=torch.bfloat16, device=DEV)
        fc.fc_qkv_project_scatter(handle, 0, x, w, bias, 0, A, None, q)
        k, v = torch.empty((1, Hkv, A, Dh), dtype=torch.bfloat16, device=DEV), torch.empty((1, Hkv, A, Dh), dtype=torch.bfloat16, device=DEV)
        fc.fc_cache_read_rows(handle, 0, k, v, 0, A)
        torch.cuda.synchronize()
        fc.fc_cache_free(handle)
        got.append((q, k, v))
    assert torch.isfinite(got[0][0].float()).all()
    for a, b in zip(*got):
        assert torch.equal(a, b)


# hidden 1088: in step; 2048: rotated starts (not where the hidden dimension is in parts)
LAYERS = [(shape, mode, K, N) for shape in sorted(ROWS) for mode, shapes in (("gated", ROWS), ("residual", (0, 1, 2, 3, 9, 10)), ("parts", (0, 1, 2, 9, 10)))
          for K, N in ((1088, 31232), (2048, 16640)) if shape in shapes and (mode, K) != ("parts", 2048)]


@pytest.mark.parametrize("shape,mode,K,N", LAYERS)
def test_layer_in_every_tile_shape(shape, mode, K, N, knob):
    """Whole matrices (four of them exceed the memory-side cache) and by halves of their outputs (four do not)."""
    print("[case] read once, layer, shape", shape, mode, K, N, flush=True)
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    knob("FC_LIN_KSPLIT", "3" if mode == "parts" else "1")
    M, gated = ROWS[shape], mode == "gated"
    n = N // 2 if gated else N
    gen = torch.Generator(device=DEV).manual_seed(shape)
    w = torch.empty((n, K), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    aux = torch.empty((n, K) if gated else (M, n), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02 if gated else 1.0, generator=gen)
    x = torch.empty((M, K), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    ws = torch.empty(16 + 3 * M * n * 4, dtype=torch.uint8, device=DEV)

    def run(lo, hi):
        out = torch.full((M, hi - lo), float("nan"), dtype=torch.bfloat16, device=DEV)
        if gated:
            fc.fc_ffn_gate_up("bf16", x, w[lo:hi], aux[lo:hi], M, K, hi - lo, out, ws)
        else:
            fc.fc_linear_residual("bf16", x, w[lo:hi], aux[:, lo:hi].contiguous(), M, K, hi - lo, out, ws)
        torch.cuda.synchronize()
        return out

    whole, halves = run(0, n), torch.cat([run(0, n // 2), run(n // 2, n)], 1)
    assert torch.isfinite(whole.float()).all()
    if K % 2048 != 0:
        assert torch.equal(whole, halves)
    else:
        # (starts along the hidden dimension go by the number of tiles: sums in another order, one result in some ten rounded the
        # other way, by 2^-8: 2^-8 sqrt(0.1) = 1.2e-3)
        a, b = whole.float(), halves.float()
        assert (a - b).norm() <= 2e-3 * b.norm()


@pytest.mark.parametrize("K", [2112, 2048])
@pytest.mark.parametrize("shape", [0, 1, 3, 9])
def test_vocabulary_in_every_tile_shape(shape, K, knob):
    print("[case] read once, vocabulary, shape", shape, K, flush=True)
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    M, V = ROWS[shape], 65664
    assert 2 * K * V > 256 << 20
    gen = torch.Generator(device=DEV).manual_seed(shape)
    w = torch.empty((V, K), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    x = torch.empty((M, K), dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
    ws = torch.empty(fc.fc_lm_head_workspace_bytes("bf16", M, K, V), dtype=torch.uint8, device=DEV)
    tok, conf = torch.full((M,), -5, dtype=torch.int32, device=DEV), torch.full((M,), float("nan"), device=DEV)
    fc.fc_lm_head_argmax("bf16", x, w, M, K, V, tok, conf, ws)
    z = torch.cat([x.double() @ w[i:i + 16416].double().T for i in range(0, V, 16416)], 1)
    top, second = z.topk(2, 1)[0].T
    # fp32 sums of 2048 products: the logits are 4 at most, 2^-22 apart; some thirty additions of that size
    assert torch.equal(tok.long()[top - second > 1e-5], z.argmax(1)[top - second > 1e-5])
    assert torch.allclose(conf.double(), 1.0 / torch.exp(z - top[:, None]).sum(1), rtol=1e-5, atol=0.0)
