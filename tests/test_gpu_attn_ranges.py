"""The attention kernel that cuts the keys into ranges, in every workgroup shape: stages that are whole, partial, few and many, and
rows whose scores rise so far behind the first keys that they are computed again with the exact maximum."""
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
