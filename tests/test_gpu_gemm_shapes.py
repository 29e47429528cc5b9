"""GPU parity of the tiled GEMM's 256 x 256 tile (two slabs, one wave per SIMD) and of problems
cut into two launches, at the edges: an odd number of slabs, ragged rows, one and few stages, parts of the
hidden dimension."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import fc_oracle as orc
from paper_2505_21467_amd import binding as fc
from paper_2505_21467_amd import inputs
from tests import test_gpu_read_once
from tests.harness import assert_close
from tests.test_gpu_parity import _compare_cache, _pair
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


@pytest.mark.parametrize("shape", [5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("M,K,N", [(5, 256, 256), (64, 320, 384), (65, 256, 1152), (130, 448, 640)])
def test_few_row_tiles(shape, M, K, N, knob):
    """64 or 128 rows per tile: ragged rows, one tile and several, dealt pairs that end inside a tile."""
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    _linear(M, K, N, True, "gated, shape %d" % shape)
    if shape >= 9 and M > 32:
        _linear(M, K, N, False, "linear, shape %d" % shape)
        knob("FC_LIN_KSPLIT", "2")
        if K >= 512 or shape == 9:
            _linear(M, 512, N, False, "linear in parts, shape %d" % shape)
    if shape == 9:
        x, w = inputs.normal(22, "x", (M, K), 1.0, "bf16"), inputs.normal(22, "w", (N, K), 0.03, "bf16")
        _check_lm_head("bf16", x, w, "vocabulary, shape 9")


@pytest.mark.parametrize("M,K,N", [(16, 4096, 7680), (16, 4096, 7616), (32, 3584, 6400), (9, 3584, 13312)])
def test_few_rows_gated_on_both_sides_of_the_line(M, K, N):
    """Tiled GEMM in half slabs (240, 238 and 200 of them), slabs (208)."""
    _linear(M, K, N, True, "gated, few rows")


@pytest.mark.parametrize("K,N", [(3584, 9216), (3584, 9152), (4096, 6400), (4096, 6336)])
def test_few_rows_gated_by_dealt_pairs_and_at_hidden_4096(K, N):
    """192 tiles of 48 dealt pairs: tiled GEMM, 191: whole-row kernel; 200 half slabs: tiled GEMM, 198: whole-row kernel."""
    _linear(11, K, N, True, "gated, few rows")


@pytest.mark.parametrize("shape", [1, 2, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("M,K,N", [(33, 2048, 128), (64, 2048, 1152), (61, 4096, 384), (128, 2048, 640)])
def test_start_along_the_hidden_dimension(shape, M, K, N, knob):
    """Weight rows a multiple of 4 KB apart: each workgroup starts at a stage of its own (one row tile), one unit and several,
    fewer and more units than stages."""
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    _linear(M, K, N, True, "gated, shape %d" % shape)
    if shape < 5 or shape >= 9:
        _linear(M, K, N, False, "linear, shape %d" % shape)
        knob("FC_LIN_KSPLIT", "1")  # (so few outputs are cut along the hidden dimension otherwise)
        _linear(M, K, N, False, "linear in one part, shape %d" % shape)
    if shape in (1, 9):
        x, w = inputs.normal(24, "x", (M, K), 1.0, "bf16"), inputs.normal(24, "w", (N, K), 0.01, "bf16")
        _check_lm_head("bf16", x, w, "vocabulary, shape %d" % shape)


@pytest.mark.parametrize("shape,M,K,units", [(9, 33, 2048, 257), (9, 64, 2048, 520), (1, 128, 4096, 264), (10, 40, 2048, 258), (7, 61, 2048, 300)])
def test_start_along_the_hidden_dimension_beyond_one_round(shape, M, K, units, knob):
    """The same by the place of a workgroup among 256: one and two units more than a round, two rounds and eight."""
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    if shape in (1, 9):
        print("[case] vocabulary", shape, M, K, units, flush=True)
        x, w = inputs.normal(25, "x", (M, K), 1.0, "bf16"), inputs.normal(25, "w", (128 * units, K), 0.01, "bf16")
        _check_lm_head("bf16", x, w, "vocabulary, shape %d" % shape)
    else:
        _linear(M, K, {7: 48 * 64 * (units // 64 + 1), 10: 32 * units}[shape], True, "gated, shape %d" % shape)


@pytest.mark.parametrize("V", [26624, 26496])
def test_few_rows_vocabulary_on_both_sides_of_the_line(V):
    """208 slabs: tiled GEMM; 207: runs of entries."""
    print("[case] vocabulary", V, flush=True)
    x, w = inputs.normal(23, "x", (5, 3584), 1.0, "bf16"), inputs.normal(23, "w", (V, 3584), 0.03, "bf16")
    _check_lm_head("bf16", x, w, "vocabulary of %d" % V)


@pytest.mark.parametrize("shape", [1, 2, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("B,d,Hq,Hkv,A", [(3, 192, 8, 2, 23), (1, 64, 3, 1, 65), (2, 320, 4, 4, 160), (1, 2048, 4, 2, 63)])
def test_few_row_tiles_projection(shape, B, d, Hq, Hkv, A, knob):
    print("[case] projection, shape", shape, B, d, Hq, Hkv, A, flush=True)
    knob("FC_PROJ_GEMM_SHAPE", str(shape))
    dtype, L = "bf16", 40
    w, S = inputs.Workload("t", dtype, B, d, Hq, Hkv, 128, L, A), L + A
    g, o = _pair(dtype, B, d, Hq, Hkv, 128, S + 5, max_rows=A, fill=-0.75)
    K, V = inputs.kv_fill(w, 11, L)
    g.write_rows(0, K, V, 0)
    o.write_rows(K, V, 0)
    W, b, X = inputs.weights(w, 11), inputs.bias(w, 11), inputs.hidden_states(w, 11, A)
    Qg, Og = g.step(0, X, W, b, L, S)
    Qo, Oo = o.step(X, W, b, L, S)
    assert_close(Qg, Qo, dtype, "Q")
    assert_close(Og, Oo, dtype, "O")
    written = np.zeros((B, S + 5), bool)
    written[:, L:S] = True
    _compare_cache(g, o, dtype, written=written, what="projection")
    g.close()


# Value rows of the 256-row tiles: 64 consecutive positions leave in pieces of eight keys and single keys at both ends, others one by one.
@pytest.mark.parametrize("shape", [0, 3, 4])
@pytest.mark.parametrize("B,L,A,listed", [
    (1, 40, 64, False),   # whole pieces only
    (2, 43, 131, False),  # off a multiple of eight, across a tile of 64 keys; the second sequence begins inside a step
    (1, 0, 80, False),    # a last step of 16 rows, the fewest that are taken in pieces
    (1, 5, 79, False),    # and of 15
    (3, 61, 192, False),  # every step one sequence's, two row tiles
    (1, 1, 86, False),    # a last step of 22 with seven single keys at either end, more than eight
    (2, 33, 128, True),   # lists: a step of consecutive positions, one with gaps, padded rows
])
def test_value_rows_of_the_wide_tiles(shape, B, L, A, listed, knob):
    print("[case] value rows, shape", shape, B, L, A, listed, flush=True)
    knob("FC_PROJ_GEMM_SHAPE", str(shape))
    dtype, d, Hq, Hkv = "bf16", 128, 4, 2  # the first value slab lies inside a wave's 40 dealt pairs
    S = L + (2 * A if listed else A)
    w = inputs.Workload("t", dtype, B, d, Hq, Hkv, 128, L, A)
    g, o = _pair(dtype, B, d, Hq, Hkv, 128, S + 5, max_rows=A, fill=-0.75)
    W, b, X = inputs.weights(w, 12), inputs.bias(w, 12), inputs.hidden_states(w, 12, A)
    pos = None
    written = np.zeros((B, S + 5), bool)
    if listed:
        pos = torch.full((B, A), -1, dtype=torch.int32)
        pos[:, :64] = torch.arange(L, L + 64)
        pos[:, 64:A - 3] = torch.arange(L + 65, L + 65 + 2 * (A - 67), 2)
        for i in range(B):
            written[i, pos[i][pos[i] >= 0].numpy()] = True
    else:
        written[:, L:S] = True
    Qg = g.project(0, X, W, b, L, pos=pos)
    Qo = o.project_only(X, W, b, L, pos=pos)
    assert_close(inputs.as_oracle(Qg), Qo, dtype, "Q")
    _compare_cache(g, o, dtype, written=written, what="value rows")
    g.close()


# The tile of 256 rows x 96 dealt pairs (shape 11): value rows as above, gated layers whose last run is short, and the non-temporal hint.
@pytest.mark.parametrize("B,L,A,listed", [(1, 40, 64, False), (2, 43, 131, False), (1, 5, 79, False), (3, 61, 192, False), (1, 1, 86, False), (2, 33, 128, True)])
def test_runs_of_96_pairs_projection(B, L, A, listed, knob):
    test_value_rows_of_the_wide_tiles(11, B, L, A, listed, knob)


@pytest.mark.parametrize("M,K,N", [(1, 256, 64), (255, 320, 192), (257, 1088, 320), (600, 512, 576)])
def test_runs_of_96_pairs_gated(M, K, N, knob):
    knob("FC_LIN_WIDE_SHAPE", "11")
    _linear(M, K, N, True, "gated, shape 11")


@pytest.mark.parametrize("K", [1088, 1024])
def test_runs_of_96_pairs_read_once(K, knob, monkeypatch):
    monkeypatch.setitem(test_gpu_read_once.ROWS, 11, 200)
    test_gpu_read_once.test_projection_in_every_tile_shape(11, K, knob)


@pytest.mark.parametrize("M,N,gated", [
    (20, 296 * 64, True),      # few rows of a wide layer, where the tiled GEMM takes over from the whole-row kernel
    (1200, 53 * 128, False),   # the last two slabs in a second launch
    (1800, 36 * 128, False),   # the last eight rows in a second launch
    (512, 296 * 64, True),     # 474 tiles of 80 dealt pairs, in one launch
    (1024, 296 * 64, True),    # 256 gated slabs in the 256 x 256 tile, 40 in a smaller one
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


@pytest.mark.parametrize("M,K,N,gated", [
    (5, 3584, 1, False), (1, 1536, 1003, True),        # fewer outputs than workgroups: one workgroup, runs of three and four
    (17, 2048, 1023, False), (33, 1536, 1027, False),  # runs of three and four, four and five; two and three tiles of rows
    (96, 1536, 4097, False), (80, 2560, 4352, False),  # runs of 16 and 17: two weight tiles
    (96, 2048, 4096, True), (48, 3072, 4160, True),    # pairs of 16 at six tiles of rows; two weight tiles at three
    (64, 4096, 1024, False), (32, 4096, 8192, False),  # workgroups start at eight stages; runs of 32
    (20, 512, 8192, True), (3, 8192, 264, False),
    (256, 2048, 2048, False), (200, 1536, 1000, False),  # four tiles of 64 rows; several tiles, the last ragged
    (130, 2048, 4096, False), (65, 1536, 4100, False),   # three tiles, runs of 51 and 52; two tiles, runs of 32 and 33
    (97, 1536, 2050, True), (128, 1536, 4096, True),     # pairs in runs of 25 and 26, and of 32
    (7, 3584, 8200, False),                            # one output quad too many: whole-row kernel
    (33, 512, 2753, False), (34, 512, 4225, False),    # tiles of 48 rows, one and two weight tiles
    (36, 512, 2243, True), (148, 1024, 1153, True),    # gated: tiles of 48 and of 64 rows, runs of up to 16
])
def test_layers_of_few_outputs(M, K, N, gated):
    """Ends of the runs, of the tiles of window rows and of the covered range."""
    _linear(M, K, N, gated, "few outputs")
    if not gated:  # without a residual
        x, w = inputs.normal(2, "x", (M, K), 1.0, "bf16"), inputs.normal(2, "w", (N, K), 0.05, "bf16")
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        ws = torch.empty(max(16, fc.fc_linear_workspace_bytes("bf16", M, K, N)), dtype=torch.uint8, device=DEV)
        fc.fc_linear_residual("bf16", x.to(DEV), w.to(DEV), None, M, K, N, out, ws)
        ref = orc.linear_residual(inputs.as_oracle(x), inputs.as_oracle(w), None, "bf16")
        assert_close(inputs.as_oracle(out), ref, "bf16", "few outputs, no residual")


@pytest.mark.parametrize("M,K,V", [
    (1, 512, 2), (15, 2560, 1721), (17, 3584, 33), (32, 512, 4097), (9, 1536, 8193), (32, 512, 16385), (31, 3584, 4095), (5, 4096, 300), (2, 512, 16384),
])
def test_small_vocabulary(M, K, V):
    """Runs of one to 64 entries, one to four weight tiles, fewer entries than parts; 16385: one too many, runs in passes."""
    print("[case] vocabulary", M, K, V, flush=True)
    x, w = inputs.normal(25, "x", (M, K), 1.0, "bf16"), inputs.normal(25, "w", (V, K), 0.03, "bf16")
    _check_lm_head("bf16", x, w, "small vocabulary of %d" % V)


# The hidden dimension in parts, every tile shape that has them: an odd number of slabs, ragged rows, parts of unequal numbers of stages.
@pytest.mark.parametrize("shape,parts", [(0, 3), (1, 2), (2, 5), (3, 2), (3, 7), (9, 16), (10, 4)])
@pytest.mark.parametrize("M,K,N", [(300, 4160, 384), (33, 4096, 128)])
def test_parts_of_every_shape(shape, parts, M, K, N, knob):
    knob("FC_LIN_WIDE_SHAPE", str(shape))
    knob("FC_LIN_KSPLIT", str(parts))
    _linear(M, K, N, False, "shape %d in %d parts" % (shape, parts))


# Layers that are cut where there is space for the partial sums, and run uncut where a call brings only what it must.
@pytest.mark.parametrize("M,K,N", [(480, 8192, 3072), (600, 6144, 3584), (700, 8192, 2048)])
def test_parts_as_the_space_allows(M, K, N):
    print("[case] parts by space", M, K, N, flush=True)
    x, w, r = inputs.normal(4, "x", (M, K), 1.0, "bf16"), inputs.normal(4, "w", (N, K), 0.05, "bf16"), inputs.normal(4, "r", (M, N), 1.0, "bf16")
    xd, wd, rd = x.to(DEV), w.to(DEV), r.to(DEV)
    ref = orc.linear_residual(inputs.as_oracle(x), inputs.as_oracle(w), inputs.as_oracle(r), "bf16")
    useful = fc.fc_linear_workspace_bytes("bf16", M, K, N)
    assert useful > 0 and useful % (4 * M * N) == 0
    ws = torch.empty(useful, dtype=torch.uint8, device=DEV)
    for space, n in ((ws, useful), (ws, useful - 1), (None, 0)):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        fc.fc_linear_residual("bf16", xd, wd, rd, M, K, N, out, space, n)
        torch.cuda.synchronize()
        assert_close(inputs.as_oracle(out), ref, "bf16", "%d bytes of workspace" % n)


def _launches(call):
    """(workgroups, threads of one) of every kernel that `call(stream)` enqueues, from a captured graph that is not run."""
    class Params(ctypes.Structure):  # hipKernelNodeParams
        _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                    ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]
    call(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        call(stream.cuda_stream)
    hip = ctypes.CDLL("libamdhip64.so")
    raw, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = Params()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        out.append((p.grid[0], p.block[0]))
    return out


# One round of 256 x 96-pair tiles, above 512 rows too and at hidden sizes above 4096, where tiles of 64 rows are not taken.
@pytest.mark.parametrize("M,K,slots", [(740, 4608, 108), (558, 6144, 108), (740, 4096, 108)])
def test_runs_of_96_pairs_where_they_fill_a_round(M, K, slots):
    print("[case] 96 pairs", M, K, slots, flush=True)
    x, w, o = (torch.zeros(s, dtype=torch.bfloat16, device=DEV) for s in ((M, K), (slots * 64, K), (M, slots * 64)))
    got = _launches(lambda s: fc.fc_ffn_gate_up("bf16", x, w, w, M, K, slots * 64, o, None, 0, s))
    assert got == [(72 * 3, 256)], got
