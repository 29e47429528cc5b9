"""The attention kernel that cuts the keys into ranges, in every workgroup shape: stages that are whole, partial, few and many, and
rows whose scores rise behind the first keys, so that their reference maxima move."""
import pytest
import torch

from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs
from tests.harness import GpuLayerCache, OracleLayerCache, assert_close

SHAPES = ["8,4", "4,4", "2,4", "8,8", "4,8"]


def _case(B, Hq, Hkv, A, S, change=lambda K, V: None, pad=True):
    from oracle import fc_oracle as orc
    dt, Dh = "bf16", 128
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 70, max_rows=max(A, 64), fill=float("nan"))  # keys past kv_len are not numbers
    o = OracleLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 70)
    K, V = inputs.kv_fill(w, 2, S)
    change(K, V)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, Hq, A, Dh), 1.0, dt)
    pos = inputs.window_positions(B, 0, A)
    if pad:
        pos[B - 1, A // 2] = -1  # a padded row: zeros
    ref = orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, inputs.as_oracle(pos))
    return g, g.dev_t(Q), pos, ref


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
@pytest.mark.parametrize("S,wgs", [(1, 1), (31, 1), (33, 1), (64, 1), (65, 1), (190, 1), (256, 1), (257, 1), (300, 1), (331, 1), (640, 1),
                                   (257, 1000), (703, 1000), (1400, 24)])
def test_stages_whole_partial_few_and_many(tiles, S, wgs, knob):
    """One range (1 .. 10 stages: fewer than the ring has, as many, more) and several; the last with 1 .. 64 keys."""
    print("[case] ranges", tiles, S, wgs, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", wgs)
    g, Q, pos, ref = _case(2, 6, 2, 23, S)
    p = fc.fc_attention_plan(g.cfg, 23, S)
    assert (p["kind"], p["tiles_per_wg"], p["waves"]) == (1, *map(int, tiles.split(","))) and (p["splits"] > 1) == (wgs > 1 and S > 128)
    O = g.attend(0, Q, S, pos)
    assert_close(inputs.as_oracle(O), ref, "bf16", tiles)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
@pytest.mark.parametrize("S,wgs", [(331, 1), (1400, 24)])
def test_scores_that_rise_behind_the_first_keys(tiles, S, wgs, knob):
    """Keys 60 times as long behind the first 40: scores of several hundred nats, so that weights relative to the first keys overflow.
    The weights are then all but one-hot and the bound is that of the rounded result."""
    print("[case] rising scores", tiles, S, wgs, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", wgs)

    def change(K, V):
        K[:, :, 40:] = (K[:, :, 40:].float() * 60).to(K.dtype)
    g, Q, pos, ref = _case(2, 6, 2, 23, S, change)
    O = g.attend(0, Q, S, pos)
    assert torch.isfinite(O.float()).all()
    assert_close(inputs.as_oracle(O), ref, "bf16", tiles)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
def test_large_values_behind_a_low_first_maximum(tiles, knob):
    """Scores some 30 nats above the first keys' and values of 1e30: the sums of weights are finite, weights times values are not, the result
    is.  The result scales with the values exactly: compared at values of 1."""
    print("[case] large values", tiles, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", 1)
    S, scale = 331, 2.0 ** 100

    def low(K, V):
        K[:, :, :40] = 0
        K[:, :, 40:] = (K[:, :, 40:].float() * 12).to(K.dtype)

    def change(K, V):
        low(K, V)
        V[:] = (V.float() * scale).to(V.dtype)
    g, Q, pos, ref = _case(2, 6, 2, 23, S, low)
    small = g.attend(0, Q, S, pos)
    assert_close(inputs.as_oracle(small), ref, "bf16", tiles)
    g.close()
    g, Q, pos, _ = _case(2, 6, 2, 23, S, change)
    large = g.attend(0, Q, S, pos)
    assert torch.isfinite(large.float()).all()
    assert_close(inputs.as_oracle((large.float() / scale).to(large.dtype)), ref, "bf16", tiles)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
@pytest.mark.parametrize("S,wgs", [(640, 1), (1400, 24)])
def test_peaked_weights_lose_no_more_than_rounding(tiles, S, wgs, knob):
    """Scores of deviation 4: one key or a few carry a row.  The sum is of the rounded weights, so the rounding of the largest cancels.  Bound of
    the relative error: the rounded result 1.7e-3, and a weight's share at most 1.2e-3 beside it (2^-9 / sqrt(3) of what does not cancel): 2.1e-3;
    with the sum of the weights before rounding it is 2.3e-3."""
    print("[case] peaked weights", tiles, S, wgs, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", wgs)

    def change(K, V):
        K.copy_((K.float() * 4).to(K.dtype))
    g, Q, pos, ref = _case(2, 6, 2, 23, S, change, pad=False)
    got = inputs.as_oracle(g.attend(0, Q, S, pos))
    err = float((((got - ref) ** 2).sum() / (ref ** 2).sum()) ** 0.5)
    print("error", err, flush=True)
    assert err <= 2.1e-3, err
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,A,S,bounds", [
    (1, 28, 4, 32, 9000, (2.291e-3, 2.128e-3, 1.879e-3, 1.760e-3)),
    (1, 28, 4, 32, 16800, (2.316e-3, 2.157e-3, 1.878e-3, 1.785e-3)),
    (4, 32, 32, 64, 4160, (2.336e-3, 2.245e-3, 2.046e-3, 1.953e-3)),
    (2, 28, 4, 200, 1500, (2.337e-3, 2.272e-3, 2.107e-3, 1.997e-3)),
    (8, 28, 4, 32, 2304, (2.323e-3, 2.235e-3, 2.044e-3, 1.929e-3)),
    (8, 28, 4, 256, 2304, (2.342e-3, 2.290e-3, 2.191e-3, 2.132e-3)),
])
def test_errors_of_the_plans_in_use(B, Hq, Hkv, A, S, bounds):
    """Scores of deviation 1, 2, 3, 4, the plan that a call takes, against 64 bits.  The bounds are the errors that a kernel with 32x32 tiles, whose
    references moved with every block, had on the same inputs; 0.2 % for weights that round the other way."""
    print("[case] plans in use", B, Hq, Hkv, A, S, flush=True)
    dev = torch.device("cuda:0")
    cfg = fc.make_config(1, B, 256, Hq, Hkv, 128, S, "bf16")
    assert fc.fc_attention_plan(cfg, A, S)["kind"] == 1
    handle = fc.fc_cache_alloc(cfg)
    n = fc.fc_workspace_bytes(cfg, A)
    ws = torch.empty(max(16, n), dtype=torch.uint8, device=dev)
    out = torch.empty((B, A, Hq, 128), dtype=torch.bfloat16, device=dev)
    gen = torch.Generator(device=dev)
    for deviation, bound in zip((1, 2, 3, 4), bounds):
        error = size = 0.0
        for seed in range(4 if B * A * Hq < 4000 else 2):
            gen.manual_seed(1000 * seed + S)
            K, V, Q = (torch.randn(shape, device=dev, generator=gen) for shape in ((B, Hkv, S, 128), (B, Hkv, S, 128), (B, Hq, A, 128)))
            K, V, Q = K.bfloat16(), V.bfloat16(), (Q * deviation).bfloat16()
            fc.fc_cache_write_rows(handle, 0, K, V, 0, S)
            fc.fc_active_attention(handle, 0, Q, A, S, None, out, ws, n)
            for b in range(B):
                for h in range(Hq):
                    k, v = K[b, h // (Hq // Hkv)].double(), V[b, h // (Hq // Hkv)].double()
                    ref = torch.softmax(Q[b, h].double() @ k.t() / 128 ** 0.5, -1) @ v
                    error += float(((out[b, :, h].double() - ref) ** 2).sum())
                    size += float((ref ** 2).sum())
        error = (error / size) ** 0.5
        print("deviation", deviation, "error", error, "bound", bound, flush=True)
        assert error <= 1.002 * bound, (deviation, error, bound)
    torch.cuda.synchronize()
    fc.fc_cache_free(handle)


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
@pytest.mark.parametrize("S,wgs,low", [
    (331, 1, (0, 100)),       # rises in the second stage, in the middle of a block
    (331, 1, (0, 320)),       # in the last stage, which is not whole
    (1400, 24, (0, 700)),     # ranges of low references beside ranges of high ones
    (1400, 24, (700, 1400)),  # the other way round
    (1400, 1, (64, 1340)),    # high, low, high again
])
@pytest.mark.parametrize("factor,scale", [(12.0, 1.0), (60.0, 1.0), (12.0, 2.0 ** 100)])
def test_references_move(tiles, S, wgs, low, factor, scale, knob):
    """Keys of zero, then such that scores rise by some 30 or 150 nats: weights relative to the first keys would be 2^43 and more, or overflow, and times
    values of 1e30 overflow.  The result scales with the values exactly: compared at values of 1."""
    print("[case] references move", tiles, S, wgs, low, factor, scale, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", wgs)

    def change(K, V, scale=1.0):
        K.copy_((K.float() * factor).to(K.dtype))
        K[:, :, low[0]:low[1]] = 0
        V.copy_((V.float() * scale).to(V.dtype))
    g, Q, pos, ref = _case(2, 6, 2, 23, S, change)
    if scale != 1.0:
        g.close()
        g, Q, pos, _ = _case(2, 6, 2, 23, S, lambda K, V: change(K, V, scale))
    O = g.attend(0, Q, S, pos)
    assert torch.isfinite(O.float()).all()
    assert_close(inputs.as_oracle((O.float() / scale).to(O.dtype)), ref, "bf16", tiles)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", SHAPES)
@pytest.mark.parametrize("S,wgs", [(331, 1), (1400, 24)])
def test_a_row_that_is_no_number(tiles, S, wgs, knob):
    """Queries that are not numbers, in a padded row and in one that is not: zeros and NaN there, every other row the same bits."""
    print("[case] no number", tiles, S, wgs, flush=True)
    knob("FC_ATTN_TILES", tiles)
    knob("FC_ATTN_WGS", wgs)
    g, Q, pos, _ = _case(2, 6, 2, 23, S)
    good = g.attend(0, Q, S, pos).clone()
    Q[1, :, 11] = float("nan")  # the padded row
    Q[0, 2, 5] = float("nan")
    O = g.attend(0, Q, S, pos).view(2, 23, 6, 128)
    good = good.view(2, 23, 6, 128)
    assert (O[1, 11] == 0).all() and torch.isnan(O[0, 5, 2].float()).all()
    O[0, 5, 2] = good[0, 5, 2]
    assert torch.equal(O, good)
    g.close()
