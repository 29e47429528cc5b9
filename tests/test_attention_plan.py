"""The attention planner: every plan covers the keys and fits the workspace that is asked for, whatever the length up
to the cache's capacity; and every tile shape it can pick agrees with the oracle where its tiles are ragged."""
import random

import pytest

from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs
from tests.harness import GpuLayerCache, OracleLayerCache, assert_close


def test_plans_cover_the_keys_and_fit_the_workspace():
    rng = random.Random(7)
    for _ in range(300):
        hkv, g = rng.choice((1, 2, 4, 8, 32)), rng.choice((1, 2, 7, 8))
        smax, batch, rows = rng.randint(1, 20000), rng.randint(1, 8), rng.randint(1, 300)
        c = fc.make_config(1, batch, 256, hkv * g, hkv, 128, smax, "bf16")
        space = fc.fc_workspace_bytes(c, rows)
        for _ in range(6):
            a, kv = rng.randint(1, rows), rng.randint(1, smax)
            p = fc.fc_attention_plan(c, a, kv)
            assert p["splits"] * p["keys_per_split"] >= kv > (p["splits"] - 1) * p["keys_per_split"], (a, kv, p)
            if p["kind"] == 0:  # tile kernel: one round of workgroups, all keys in each
                assert p["splits"] == p["tiles_per_wg"] == 1 and p["row_tiles"] * batch * hkv <= 256 and kv <= 1200, (a, kv, p)
                continue
            assert p["keys_per_split"] % 64 == 0 and p["tiles_per_wg"] in (2, 4, 8) and p["waves"] in (4, 8)
            need = batch * hkv * p["row_tiles"] * p["splits"] * 32 * (256 + 16) if p["splits"] > 1 else 0
            assert need <= space, (a, kv, p, need, space)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,A,S", [
    (1, 2, 1, 3, 5), (1, 28, 4, 32, 96), (2, 3, 1, 100, 333),  # head dimension of V in four parts
    (2, 28, 4, 20, 300), (8, 14, 2, 16, 64), (4, 32, 32, 9, 64),  # in two; uncut (two of them full)
])
def test_short_keys_take_the_tile_kernel(B, Hq, Hkv, A, S):
    print("[case] short keys", B, Hq, Hkv, A, S, flush=True)
    from oracle import fc_oracle as orc
    Dh, dt = 128, "bf16"
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 9, max_rows=A, fill=float("nan"))  # keys past kv_len are not numbers
    o = OracleLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 9)
    assert fc.fc_attention_plan(g.cfg, A, S)["kind"] == 0
    K, V = inputs.kv_fill(w, 2, S)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, Hq, A, Dh), 1.0, dt)
    O = g.attend(0, g.dev_t(Q), S)
    assert_close(inputs.as_oracle(O), orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, None), dt, "short keys")
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("tiles", ["8,8", "4,8", "2,8", "4,4", "2,4"])
@pytest.mark.parametrize("Hq,Hkv,A,S", [(3, 1, 5, 70), (10, 2, 21, 777), (9, 1, 33, 300)])
def test_every_tile_shape_matches_oracle(tiles, Hq, Hkv, A, S, knob):
    print("[case]", tiles, Hq, Hkv, A, S, flush=True)
    knob("FC_ATTN_TILES", tiles)
    from oracle import fc_oracle as orc
    B, Dh, dt = 2, 128, "bf16"
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S, max_rows=A)
    o = OracleLayerCache(dt, B, 256, Hq, Hkv, Dh, S)
    K, V = inputs.kv_fill(w, 2, S)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, Hq, A, Dh), 1.0, dt)
    O = g.attend(0, g.dev_t(Q), S)
    assert_close(inputs.as_oracle(O), orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, None), dt, tiles)
    g.close()
