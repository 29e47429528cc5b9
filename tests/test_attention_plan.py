"""The attention planner: every plan covers the keys and fits the workspace that is asked for, whatever the length up
to the cache's capacity; and every tile shape it can pick agrees with the oracle where its tiles are ragged."""
import random

import pytest
import torch

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
            if p["kind"] != 1:  # one round of workgroups, all keys in each: the tile kernel, or the one that sums groups of keys
                assert p["splits"] == 1 and p["row_tiles"] == -(-g * a // 16), (a, kv, p)
                assert -(-p["row_tiles"] // p["tiles_per_wg"]) * batch * hkv <= 256, (a, kv, p)
            if p["kind"] == 0:
                assert p["tiles_per_wg"] == 1 and p["waves"] == 8 and kv <= 96, (a, kv, p)
                continue
            assert p["keys_per_split"] % 64 == 0
            if p["kind"] == 2:
                assert (p["tiles_per_wg"], p["waves"]) in ((1, 8), (1, 6), (2, 8)) and (p["waves"] == 8 or kv <= 1200), (a, kv, p)
                continue
            assert p["kind"] == 1 and p["tiles_per_wg"] in (2, 4, 8) and p["waves"] in (4, 8)
            need = batch * hkv * p["row_tiles"] * p["splits"] * 32 * (256 + 16) if p["splits"] > 1 else 0
            assert need <= space, (a, kv, p, need, space)


@pytest.mark.parametrize("dt,line", [("f32", 13 * 32), ("bf16", 53 * 32)])
def test_two_tiles_per_workgroup_are_cut_where_they_fill_half_a_round(dt, line):
    """128 workgroups of two tiles: in two ranges from the line on, space permitting; more workgroups: never cut."""
    for hkv, A, keys, splits in ((4, 128, line - 32, 1), (4, 128, line, 2), (4, 113, line - 31, 2), (4, 160, 16000, 1), (1, 1000, 16000, 2)):
        c = fc.make_config(1, 8 if hkv == 4 else 4, 256, hkv, hkv, 64, keys, dt)
        p = fc.fc_attention_plan(c, A, keys)
        assert (p["kind"], p["tiles_per_wg"], p["splits"]) == (0, 2, splits), (A, keys, p)
        per = -(-keys // 32 // splits) if keys % 32 == 0 else -(-(keys // 32 + 1) // splits)
        assert p["keys_per_split"] == 32 * per


@pytest.mark.gpu
@pytest.mark.parametrize("dt,A,S", [("f32", 128, 416), ("f32", 113, 449), ("bf16", 120, 1696), ("bf16", 113, 1697)])
def test_two_tiles_per_workgroup_in_two_ranges(dt, A, S):
    print("[case] two tiles", dt, A, S, flush=True)
    from oracle import fc_oracle as orc
    B, H, Dh = 8, 4, 64
    w = inputs.Workload("t", dt, B, 256, H, H, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, H, H, Dh, S + 3, max_rows=A, fill=float("nan"))  # keys past kv_len are not numbers
    o = OracleLayerCache(dt, B, 256, H, H, Dh, S + 3)
    assert fc.fc_attention_plan(g.cfg, A, S)["splits"] == 2
    K, V = inputs.kv_fill(w, 2, S)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, H, A, Dh), 1.0, dt)
    O = g.attend(0, g.dev_t(Q), S)
    assert_close(inputs.as_oracle(O), orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, None), dt, "two tiles")
    g.close()


def test_window_rows_times_heads_beyond_32_bits():
    c = fc.make_config(1, 1, 256, 256, 1, 128, 100, "bf16")
    p = fc.fc_attention_plan(c, 1 << 24, 100)  # 2^32 query rows: the split-KV kernel, not a tile kernel of no tiles
    assert p["kind"] == 1 and p["row_tiles"] == 1 << 27


def _required(pairs, g, A, kv):
    """Partial results (bytes) of one round of workgroups, tiles by the row count: what a bf16 call must bring."""
    tiles, by_len = -(-g * A // 32), max(1, -(-kv // 64) // 2)
    R = 2 if tiles <= 2 else 4 if tiles <= 7 else 8

    def nearest(target, base):
        return max(1, min((target + base // 2) // base, by_len))
    splits = nearest(256, pairs * -(-tiles // R))
    if R == 4 and pairs * -(-tiles // R) * splits < 256:
        splits = nearest(512, pairs * -(-tiles // 2))
    return pairs * tiles * splits * 32 * (256 + 16) if splits > 1 else 0


def test_calls_require_one_round_of_partial_results():
    rng = random.Random(11)
    for _ in range(300):
        hkv, g = rng.choice((1, 2, 4, 8, 32)), rng.choice((1, 2, 7, 8))
        smax, batch, rows = rng.randint(1, 20000), rng.randint(1, 8), rng.randint(1, 300)
        c = fc.make_config(1, batch, 256, hkv * g, hkv, 128, smax, "bf16")
        space = fc.fc_workspace_bytes(c, rows)
        h = fc.fc_cache_alloc(c, 0x10000, 0x10000)
        for _ in range(4):
            a, kv = rng.randint(1, rows), rng.randint(1, smax)
            need = _required(batch * hkv, g, a, kv)
            assert need <= space, (a, kv, need, space)
            if need == 0:
                continue  # (a call without workspace is accepted)
            for given in (0, need - 1):
                with pytest.raises(fc.FreeCacheError) as e:
                    fc.fc_active_attention(h, 0, 0x10000, a, kv, None, 0x10000, 0x10000 if given else None, given, 0)
                assert e.value.status == fc.FC_ERR_WORKSPACE and "%d bytes needed" % need in str(e.value)
        fc.fc_cache_free(h)
    # 28/4 heads x 16800 keys: 7 row tiles x 32 ranges at 32 rows; the most, 4 tiles x 64 ranges, at 15 .. 18 rows
    c4 = fc.make_config(1, 1, 3584, 28, 4, 128, 16800, "bf16")
    assert _required(4, 7, 32, 16800) == 4 * 7 * 32 * 8704 and fc.fc_workspace_bytes(c4, 32) == 4 * 4 * 64 * 8704
    # a workgroup per (sequence, head): nothing to merge, nothing asked for
    assert fc.fc_workspace_bytes(fc.make_config(1, 8, 4096, 32, 32, 128, 2304, "bf16"), 32) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dt,B,Hq,Hkv,Dh,A,S", [
    ("bf16", 8, 32, 32, 128, 3, 1300),   # required: nothing
    ("bf16", 1, 32, 32, 128, 14, 1563),  # one range more than required is of use
    ("f32", 1, 4, 1, 64, 8, 2000), ("bf16", 1, 6, 2, 64, 9, 3001), ("f32", 2, 2, 1, 128, 5, 700),  # no call requires any
])
def test_less_workspace_means_fewer_key_ranges(dt, B, Hq, Hkv, Dh, A, S):
    print("[case] workspace", dt, B, Hq, Hkv, Dh, A, S, flush=True)
    from oracle import fc_oracle as orc
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S, max_rows=A)
    o = OracleLayerCache(dt, B, 256, Hq, Hkv, Dh, S)
    K, V = inputs.kv_fill(w, 2, S)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, Hq, A, Dh), 1.0, dt)
    ref = orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, None)
    least = _required(B * Hkv, Hq // Hkv, A, S) if (dt, Dh) == ("bf16", 128) else 0
    full = g.ws_bytes
    for space in sorted({least, (least + full) // 2, max(least, full - 1), full, 2 * full}):
        # nothing beyond the given bytes may be written
        ws = torch.full((space + 256,), 0x5A, dtype=torch.uint8, device="cuda:0")
        O = torch.full((B, A, Hq * Dh), float("nan"), dtype=g.tdt, device="cuda:0")
        fc.fc_active_attention(g.handle, 0, g.dev_t(Q), A, S, None, O, ws if space else None, space)
        torch.cuda.synchronize()
        assert_close(inputs.as_oracle(O), ref, dt, "workspace of %d bytes" % space)
        assert bool((ws[space:] == 0x5A).all())
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,A,S", [
    (1, 2, 1, 3, 5), (1, 28, 4, 32, 96), (2, 3, 1, 100, 95),  # head dimension of V in four parts
    (2, 28, 4, 20, 63), (8, 14, 2, 16, 64), (4, 32, 32, 9, 64),  # in two
    (5, 32, 32, 9, 64), (7, 28, 4, 11, 33),  # uncut
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
@pytest.mark.parametrize("B,Hq,Hkv,A,S,per_wg,waves", [
    # 16 rows, V in four parts: a last stage of one key, of exactly a half and a whole one; one stage more than waves
    (1, 3, 1, 5, 97, 1, 8), (1, 3, 1, 6, 128, 1, 8), (1, 28, 4, 9, 1025, 1, 8), (2, 28, 4, 4, 513, 1, 8), (1, 5, 1, 7, 577, 1, 8),
    (2, 1, 1, 1, 160, 1, 8), (1, 8, 8, 33, 1300, 1, 8), (2, 3, 1, 100, 333, 1, 8),
    # in two parts; uncut, six waves
    (2, 28, 4, 20, 129, 1, 8), (2, 28, 4, 20, 300, 1, 8), (3, 28, 4, 19, 1581, 1, 8), (3, 32, 32, 8, 385, 1, 8),
    (4, 28, 4, 32, 321, 1, 6), (5, 32, 32, 3, 385, 1, 6), (2, 32, 32, 33, 769, 1, 6),
    # 32 rows, V in two parts
    (4, 28, 4, 31, 1217, 2, 8), (4, 28, 4, 29, 1281, 2, 8),
])
def test_all_keys_in_one_launch(B, Hq, Hkv, A, S, per_wg, waves):
    print("[case] one launch", B, Hq, Hkv, A, S, flush=True)
    from oracle import fc_oracle as orc
    Dh, dt = 128, "bf16"
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, A)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 70, max_rows=A, fill=float("nan"))  # keys past kv_len are not numbers
    o = OracleLayerCache(dt, B, 256, Hq, Hkv, Dh, S + 70)
    p = fc.fc_attention_plan(g.cfg, A, S)
    assert (p["kind"], p["splits"], p["tiles_per_wg"], p["waves"]) == (2, 1, per_wg, waves), p
    K, V = inputs.kv_fill(w, 2, S)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    Q = inputs.normal(2, "q", (B, Hq, A, Dh), 1.0, dt)
    pos = inputs.window_positions(B, 0, A)
    pos[B - 1, A // 2] = -1  # a padded row: zeros
    ref = orc.attend(o.cfg, inputs.as_oracle(Q), o.Kc, o.Vc, S, inputs.as_oracle(pos))
    O = g.attend(0, g.dev_t(Q), S, pos)
    assert_close(inputs.as_oracle(O), ref, dt, "one launch")
    assert not O[B - 1, A // 2].any()
    # tensors that start at an odd element, and no workspace where none is required: the same bits
    q, out = (torch.zeros(t.numel() + 1, dtype=t.dtype, device="cuda:0")[1:].view(t.shape) for t in (Q, O))
    q.copy_(Q)
    if _required(B * Hkv, Hq // Hkv, A, S) == 0:
        fc.fc_active_attention(g.handle, 0, q, A, S, pos.to("cuda:0"), out, None, 0)
    else:
        fc.fc_active_attention(g.handle, 0, q, A, S, pos.to("cuda:0"), out, g.workspace, g.ws_bytes)
    assert torch.equal(out.view(torch.int16), O.view(torch.int16))
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


@pytest.mark.gpu
def test_host_threads_with_two_shapes_share_a_cache():
    """Two threads plan and launch two shapes on one handle and stream, each with its own buffers."""
    import threading
    print("[case] two threads", flush=True)
    dt, B, Hq, Hkv, Dh, S = "bf16", 1, 14, 2, 128, 1500
    w = inputs.Workload("t", dt, B, 256, Hq, Hkv, Dh, S, 32)
    g = GpuLayerCache(dt, B, 256, Hq, Hkv, Dh, S, max_rows=32)
    g.write_rows(0, *inputs.kv_fill(w, 2, S), 0)
    stream = torch.cuda.current_stream().cuda_stream
    jobs = []
    for A, kv in ((32, S), (5, 300)):
        Q = g.dev_t(inputs.normal(A, "q", (B, Hq, A, Dh), 1.0, dt))
        O = [torch.full((B, A, Hq * Dh), float("nan"), dtype=g.tdt, device="cuda:0") for _ in range(2)]
        ws = torch.empty(max(16, fc.fc_workspace_bytes(g.cfg, A)), dtype=torch.uint8, device="cuda:0")
        fc.fc_active_attention(g.handle, 0, Q, A, kv, None, O[0], ws, ws.numel(), stream)
        jobs.append((Q, A, kv, O, ws))
    torch.cuda.synchronize()
    assert fc.fc_attention_plan(g.cfg, 32, S) != fc.fc_attention_plan(g.cfg, 5, 300)
    wrong = []

    def work(Q, A, kv, O, ws):
        try:
            for _ in range(300):
                fc.fc_active_attention(g.handle, 0, Q, A, kv, None, O[1], ws, ws.numel(), stream)
        except Exception as e:
            wrong.append(e)
    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not wrong
    for _, _, _, O, _ in jobs:
        assert torch.equal(O[0].view(torch.int16), O[1].view(torch.int16))
    g.close()
