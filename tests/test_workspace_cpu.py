"""The whole-layer workspace query promises space for every window of up to max_rows rows.  What a call must bring it says itself, when it
brings nothing."""
import re

import pytest

from paper_2505_21467_amd import binding as fc

FAKE = 0x10000  # 16-byte aligned non-NULL "device pointer"; never dereferenced on the host


def _required(cache, weights, A):
    with pytest.raises(fc.FreeCacheError) as e:
        fc.fc_full_layer_step(cache, 0, weights, FAKE, 0, A, None, 1, FAKE, None, 0, 0)
    assert e.value.status == fc.FC_ERR_WORKSPACE
    return int(re.search(r"workspace of (\d+) bytes needed", str(e.value)).group(1))


@pytest.mark.parametrize("dtype,hidden,Hq,Hkv,Dh,d_ff,B,rows", [
    ("bf16", 3584, 28, 4, 128, 18944, 1, (17, 33, 65, 181, 257, 385, 520, 900)),
    ("bf16", 3584, 28, 4, 128, 18944, 8, (5, 17, 33, 50, 65, 129)),
    ("bf16", 4096, 32, 32, 128, 12288, 1, (33, 181, 257, 600)),
    ("bf16", 4096, 32, 32, 128, 12288, 3, (11, 22, 43, 86, 171)),
    ("bf16", 5120, 40, 8, 128, 13824, 1, (33, 129, 300)),
    ("bf16", 512, 4, 2, 128, 1024, 2, (8, 9, 16, 17, 33, 200)),
    ("bf16", 2048, 16, 16, 64, 5632, 1, (33, 257, 500)),
    ("f32", 256, 4, 4, 64, 512, 4, (9, 40)),
])
def test_every_narrower_window_fits(dtype, hidden, Hq, Hkv, Dh, d_ff, B, rows):
    cfg = fc.make_config(1, B, hidden, Hq, Hkv, Dh, 2304, dtype)
    cache = fc.fc_cache_alloc(cfg, FAKE, FAKE)
    weights = fc.make_layer_weights(FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, d_ff, 1e-6)
    need = [_required(cache, weights, A) for A in range(1, max(rows) + 1)]
    for r in rows:
        got = fc.fc_full_layer_workspace_bytes(cfg, d_ff, r)
        worst = max(range(r), key=lambda a: need[a])
        assert got >= need[worst], "%d bytes for %d rows, %d needed for %d" % (got, r, need[worst], worst + 1)
    fc.fc_cache_free(cache)


@pytest.mark.parametrize("hidden,Hq,Hkv,d_ff,B", [(3584, 28, 4, 18944, 1), (3584, 28, 4, 18944, 8), (4096, 32, 32, 12288, 3), (512, 4, 2, 1024, 2)])
def test_a_wider_window_never_needs_less(hidden, Hq, Hkv, d_ff, B):
    cfg = fc.make_config(1, B, hidden, Hq, Hkv, 128, 2304, "bf16")
    got = [fc.fc_full_layer_workspace_bytes(cfg, d_ff, r) for r in range(1, 400)]
    assert got == sorted(got)
