"""GPU parity of the vocabulary kernel whose workgroups own runs of entries (bf16, at most 32 rows, runs of 64 entries and more at hidden
512, 90 at 3584 and 120 at 4096), against 64 bits: one pass and several, ragged passes and waves, 16 and 32 rows, with and without the
non-temporal hint, four orders of the chains at hidden 4096; equal logits wherever a run keeps them."""
import pytest
import torch

from paper_2505_21467_amd import binding as fc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(x, w):
    (M, K), V = x.shape, w.shape[0]
    need = fc.fc_lm_head_workspace_bytes("bf16", M, K, V)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    tok = torch.full((M,), -5, dtype=torch.int32, device=DEV)
    conf = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    fc.fc_lm_head_argmax("bf16", x, w, M, K, V, tok, conf, ws, need)
    torch.cuda.synchronize()
    return tok.long(), conf.double()


@pytest.mark.parametrize("M,K,V", [
    (1, 512, 16384), (16, 512, 16385), (17, 512, 65536), (32, 512, 65537),      # runs of 64, 64 and 65, 256, 256 and 257: a second pass
    (5, 512, 152067), (32, 512, 300001),                                      # three passes and five; with the hint
    (3, 3584, 23039), (4, 3584, 23040), (31, 3584, 23041),                    # whole-row kernel, runs of 90, of 90 and 91
    (2, 3584, 40001), (20, 3584, 40001),                                      # with the hint
    (32, 4096, 30719), (32, 4096, 30721), (9, 4096, 33001), (7, 4096, 66003), (18, 4096, 66003),  # whole-row kernel, chains in four orders, two passes
])
def test_matches_64_bits(M, K, V):
    print("[case] large vocabulary", M, K, V, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(V + M)
    w = torch.empty((V, K), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    lean = torch.randint(0, V, (M,), generator=gen, device=DEV)
    lean[0] = V - 1
    force = torch.empty((M, 1), device=DEV).uniform_(3, 12, generator=gen)
    x = (torch.empty((M, K), device=DEV).normal_(generator=gen) + force * w[lean].float()).to(torch.bfloat16)
    tok, conf = _run(x, w)
    z = torch.cat([x.double() @ w[i:i + 16384].double().T for i in range(0, V, 16384)], 1)
    top, ref_tok = z.max(1)
    ref = 1.0 / torch.exp(z - top[:, None]).sum(1)
    # fp32 sums of K products reach 20 at most: a few additions of that size, 2^-20 = 1e-6 apart, of which rms 4e-7 were seen
    assert torch.all((tok >= 0) & (tok < V))
    assert torch.all(top - z.gather(1, tok[:, None])[:, 0] <= 1e-5)
    second = z.scatter(1, ref_tok[:, None], float("-inf")).amax(1)
    clear = top - second > 1e-5
    assert torch.equal(tok[clear], ref_tok[clear])
    assert torch.allclose(conf, ref, rtol=1e-5, atol=0.0)


@pytest.mark.parametrize("M,K,V", [(11, 512, 152064), (32, 512, 152064), (16, 4096, 100002)])
def test_equal_logits_go_to_the_smaller_index(M, K, V):
    """The same weight row twice: in one lane, in two lanes, waves, passes and runs, in either order of place."""
    print("[case] equal logits", M, K, V, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(M)
    w = torch.empty((V, K), dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen)
    big = torch.empty((K,), dtype=torch.bfloat16, device=DEV).normal_(0, 0.1, generator=gen)
    x = (torch.empty((M, K), device=DEV).normal_(0, 0.1, generator=gen) + 10 * big.float()).to(torch.bfloat16)
    first, run = 100 * V // 256, 101 * V // 256 - 100 * V // 256  # of the 101st workgroup
    assert run > 256
    for places in ((first, first + 1), (first + 17, first + 22), (first + 3, first + 70), (first + 150, first + run - 1),
                   (first + run - 1, first + run), (0, V - 1), (first + 199, first + 201, first + run + 5)):
        keep = w[list(places)].clone()
        w[list(places)] = big
        tok, conf = _run(x, w)
        assert torch.all(tok == min(places)), places
        assert torch.all(conf <= 1.0 / len(places) + 1e-6)
        w[list(places)] = keep
