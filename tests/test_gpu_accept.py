"""GPU parity of the guided acceptance where its parts and its row counts have edges: vocabularies of one part, of
several and of many steps per part, one to four rows per wave and the kernel for longer blocks; ties, ranks
around topk, and a guide that agrees almost everywhere, so that long prefixes are decided by every part."""
import numpy as np
import pytest

from oracle import fc_oracle as orc
from tests.test_gpu_unmask import _gpu_accept

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,A,V", [(1, 1, 1), (2, 16, 1279), (1, 17, 1281), (2, 33, 6429), (1, 64, 5120), (1, 65, 2563), (1, 3, 200001)])
def test_long_prefixes_are_bit_exact(B, A, V):
    print("[case]", B, A, V, flush=True)
    rng = np.random.default_rng(A * 131 + V)
    MASK, L = 300000, 2 * A
    for topk, tau, noise, ties in ((1, 0.0, 0.02, False), (2, 0.5, 0.1, True), (8, 0.0, 0.4, False), (3, 1.0, 0.1, True)):
        topk = min(topk, V)
        dlm = rng.normal(0, 3, (B, A, V)).astype(np.float32)
        ar = (dlm + rng.normal(0, noise, (B, A, V))).astype(np.float32)
        if ties:
            dlm, ar = np.round(dlm), np.round(ar)
        pos = np.stack([np.sort(rng.choice(L, A, replace=False)) for _ in range(B)]).astype(np.int32)
        tokens = np.full((B, L), MASK, np.int32)
        tokens[rng.random((B, L)) < 0.2] = 0
        want_t = tokens.copy()
        want = orc.guided_accept(dlm, ar, pos, topk, tau, MASK, want_t)
        got_t, n, pn, cn = _gpu_accept(dlm, ar, pos, 0, topk, tau, MASK, tokens)
        assert np.array_equal(n, want[0]) and np.array_equal(got_t, want_t)
        assert np.array_equal(pn, want[1]) and np.array_equal(cn, want[2])


@pytest.mark.parametrize("V", [777, 5124, 20487])
@pytest.mark.parametrize("A", [5, 33, 66])
def test_entries_ahead_of_the_token_wherever_they_lie(A, V):
    """topk - 1 and topk entries of the guide ahead of the proposed token: around it, spread over the row, at the proposal's next
    best entries, tied with it on either side, and a token whose guide value is the lowest there is."""
    rng = np.random.default_rng(A * 7 + V)
    MASK, L = 300000, A + 2
    pos = np.arange(A, dtype=np.int32)[None]
    for topk in (1, 2, 3, 8):
        dlm = rng.normal(0, 1, (1, A, V)).astype(np.float32)
        ar = rng.normal(0, 1, (1, A, V)).astype(np.float32)
        for a in range(A):
            t = int(rng.integers(20, V - 20))
            n = topk - 1 if a + 1 < A else topk  # the last row does not match
            order = np.argsort(-dlm[0, a])
            where = (a + topk) % 5
            if where == 0:
                at = t + 1 + np.arange(n)
            elif where == 1:
                at = rng.choice(np.delete(np.arange(V), t), n, replace=False)
            elif where == 2:
                at = order[order != t][:n]
            elif where == 3:
                at = t - 1 - np.arange(n)
            else:
                at = t + 2 + 2 * np.arange(n)
            dlm[0, a, t] = 50.0
            ar[0, a, t] = 9.0
            ar[0, a, at] = 9.0 if where == 3 else 10.0 + rng.random(n)  # smaller ids: ties count
            if where == 4:
                ar[0, a, t + 1] = 9.0  # a tie behind it does not
                if a + 1 == A:
                    ar[0, a] = -np.inf  # and here every entry ties
        tokens = np.full((1, L), MASK, np.int32)
        want_t = tokens.copy()
        want = orc.guided_accept(dlm, ar, pos, topk, 0.0, MASK, want_t)
        assert want[0][0] == A - 1
        got_t, k, pn, cn = _gpu_accept(dlm, ar, pos, 0, topk, 0.0, MASK, tokens)
        assert np.array_equal(k, want[0]) and np.array_equal(got_t, want_t)
        assert np.array_equal(pn, want[1]) and np.array_equal(cn, want[2])


@pytest.mark.parametrize("V,parts", [(2097152, 0), (131072, 8), (140003, 8)])
def test_many_entries_of_one_record_ahead_of_the_token(V, parts, knob):
    """Records of 65536 entries and more (parts: asked for by the tuning knob), read again for topk 3 and 8: so many entries ahead of
    the proposed token, or tied with it, that a lane of the wave meets 1024 of them, and just topk - 1, topk and topk + 1 in
    one lane.  Behind the row under test one that matches: two accepted, or one."""
    print("[case]", V, parts, flush=True)
    from paper_2505_21467_amd import binding as fc
    B, A, MASK, L, REC = 9, 2, 3000000, 2, 65536
    if parts:
        knob("FC_ACCEPT_WGS", str(parts * B * A))
    assert fc.fc_guided_accept_workspace_bytes(B, A, V) == B * A * (8 + 16 * (parts or 128))
    pos = np.arange(A, dtype=np.int32)[None].repeat(B, 0)
    for topk in (2, 3, 8):
        dlm = np.zeros((B, A, V), np.float32)
        ar = np.full((B, A, V), -1.0, np.float32)
        expect = []
        for b in range(B):
            t = V - 5 if b != 1 else 3  # in the last record, or in the first
            dlm[b, 0, t], ar[b, 0, t] = 50.0, 9.0
            dlm[b, 1, 7], ar[b, 1, 7] = 50.0, 9.0
            lane = 11  # entries 11, 75, ... are one lane's
            if b == 0:
                ar[b, 0, :REC] = 10.0
            elif b == 1:
                ar[b, 0, -REC:] = 10.0
            elif b == 2:
                ar[b, 0, :REC] = 9.0  # smaller ids: ties count
            elif b == 3:
                ar[b, 0, lane:REC:64] = 10.0
            elif b == 4:
                ar[b, 0, :REC // 2] = 10.0
            else:
                n = topk - 1 + (0, 1, 2, 0)[b - 5]
                ar[b, 0, lane:lane + 64 * n:64] = 10.0 if b < 8 else 9.0
            expect.append(2 if b in (5, 8) else 1)
        tokens = np.full((B, L), MASK, np.int32)
        want_t = tokens.copy()
        want = orc.guided_accept(dlm, ar, pos, topk, 0.0, MASK, want_t)
        assert list(want[0]) == expect
        got_t, n, pn, cn = _gpu_accept(dlm, ar, pos, 0, topk, 0.0, MASK, tokens)
        assert np.array_equal(n, want[0]) and np.array_equal(got_t, want_t), (topk, n, want[0])
        assert np.array_equal(pn, want[1]) and np.array_equal(cn, want[2])
