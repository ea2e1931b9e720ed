"""Verification at the edges of its row slices: 8, 16 and 32 slices per row,
vocabularies with empty slices and with slices longer than one walk of the
draw, masked (-inf) logits, draws at both ends, a residual of no weight."""
import numpy as np
import pytest
import torch

from oracle import verify_tree_greedy
from synth import SMALL_BF16_CHAIN, make_verify_tree_targets
from test_gpu_verify import run_chain_verify

pytestmark = pytest.mark.gpu


# rows = B (2 K + 1) sampled, B (K + 1) greedy: up to 32 rows take 32 slices,
# up to 64 take 16; 16 ids: 4 per slice and 28 empty slices; 262144 ids: 8192
# per draw slice, two walks of 4096
@pytest.mark.parametrize("T", [0.0, 0.7])
@pytest.mark.parametrize("vocab,B,K", [(16, 3, 2), (16, 40, 4), (4096, 1, 1), (4112, 4, 6), (5008, 10, 6),
                                       (262144, 2, 2), (128256, 1, 63)])
def test_verify_chain_slices(vocab, B, K, T):
    cfg = SMALL_BF16_CHAIN.with_(vocab=vocab, batch=min(B, 64), n_steps=K, n_sets=1, f_map=(0,) * K)
    run_chain_verify(cfg, B, K, T, seed=11)


def _call(dr, tl, toks, T, dl, u):
    out = dr.verify_chain(tl, toks, T, dl, u)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    return out["n"].tolist(), out["next"].tolist()


@pytest.mark.parametrize("vocab", [4112, 128256])
def test_verify_chain_masked_and_extreme_draws(vocab):
    """Most ids masked with -inf (whole slices of them): statistics and draws
    come from the others; u = 0 gives the first id of positive weight, u = 1
    the last; equal rows leave no residual."""
    from paper_2602_01762_amd import Drafter
    B, K = 4, 2
    dr = Drafter(SMALL_BF16_CHAIN.with_(vocab=vocab, batch=B, n_steps=K, n_sets=1, f_map=(0, 0)))
    live = [vocab - 5, vocab // 2, vocab // 2 + 1, 7]
    tl = torch.full((B, K + 1, vocab), float("-inf"), device="cuda")
    tl[:, :, live] = torch.tensor([1.0, 0.5, 2.0, 0.25], device="cuda")
    dl = tl[:, :K].contiguous()
    toks = torch.full((B, K), vocab // 2, dtype=torch.int32, device="cuda")
    # greedy: the largest live id's value wins; the first draft is not it
    n, nxt = _call(dr, tl, toks, 0.0, None, None)
    assert n == [0] * B and nxt == [vocab // 2 + 1] * B
    # sampled, equal rows: every draft kept (ratio 1), the extra token by u
    u = torch.tensor([[0.1, 0.9, 0.0], [0.1, 0.9, 1.0], [0.0, 0.0, 0.5], [0.5, 0.5, 0.999999]], device="cuda")
    n, nxt = _call(dr, tl, toks, 1.0, dl, u)
    w = np.exp(np.array([0.25, 0.5, 2.0, 1.0]))
    cdf, ids = np.cumsum(w) / w.sum(), [7, vocab // 2, vocab // 2 + 1, vocab - 5]
    want = [ids[min(3, int(np.searchsorted(cdf, x, side="right")))] for x in (0.0, 1.0, 0.5, 0.999999)]
    assert n == [K] * B and nxt == want
    # u = 1 rejects the first draft although the rows are equal: no residual
    # is left, so the draw comes from the target row
    n, nxt = _call(dr, tl, toks, 1.0, dl, torch.ones_like(u))
    assert n == [0] * B and nxt == [vocab - 5] * B
    # a row of -inf alone: greedy takes its lowest id
    n, nxt = _call(dr, torch.full_like(tl, float("-inf")), toks, 0.0, None, None)
    assert n == [0] * B and nxt == [0] * B
    # a draft outside the vocabulary is not kept; the draw is the target's
    toks[1, 0] = vocab
    out = dr.verify_chain(tl, toks, 1.0, dl, u)
    torch.cuda.synchronize()
    assert dr.device_status() == -1
    assert out["n"].tolist() == [K, 0, K, K] and out["next"].tolist() == want
    dr.close()


@pytest.mark.parametrize("B,nodes", [(1, 1), (1, 40), (2, 30), (4, 64)])
def test_verify_tree_slices(B, nodes):
    from paper_2602_01762_amd import Drafter
    V = 5008
    dr = Drafter(SMALL_BF16_CHAIN.with_(vocab=V, batch=4))
    rng = np.random.default_rng(nodes)
    parent = np.array([[int(rng.integers(-1, j)) if j else -1 for j in range(nodes)] for _ in range(B)], np.int32)
    toks = rng.integers(0, V, (B, nodes)).astype(np.int32)
    tk, pa = torch.tensor(toks, device="cuda"), torch.tensor(parent, device="cuda")
    tl = make_verify_tree_targets(tk, pa, V, seed=nodes)
    out = dr.verify_tree(tl, tk, pa)
    torch.cuda.synchronize()
    for b in range(B):
        ref = verify_tree_greedy(tl[b].cpu().numpy().astype(np.float64), toks[b], parent[b])
        assert (int(out["n"][b]), int(out["next"][b])) == (ref["n"], ref["next"])
        assert out["path"][b].tolist()[:ref["n"]] == ref["path"]
    dr.close()
