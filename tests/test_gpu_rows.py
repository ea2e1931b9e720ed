"""Passes of more rows than the 16-row-tile kernels take (bf16): the tile
kernel at the edges of its row and feature tiles, and the two routes that
read feature rows once instead of per row, against the oracle."""
import numpy as np
import pytest
import torch

from harness import LOGIT_TOL, check_chain, check_draft_kv, gpu_setup, log, oracle_for
from synth import SMALL_BF16_CHAIN, host_inputs, host_weights, make_inputs, make_weights, scoring_target

pytestmark = pytest.mark.gpu


# accepted rows in all: one past the small kernels, whole and one past a
# 64- and a 128-row tile, two chunks of a long front; hidden 480: no
# embedding table, so the staged operand and the whole QKV product
@pytest.mark.parametrize("batch,n,hidden", [(1, 65, 512), (2, 64, 512), (3, 43, 512), (1, 193, 512),
                                            (1, 2049, 512), (1, 129, 480), (5, 53, 480)])
def test_catchup_row_tiles(batch, n, hidden):
    cfg = SMALL_BF16_CHAIN.with_(name="small_catchup_%dx%d_h%d" % (batch, n, hidden), batch=batch,
                                 n_new=(n, n), ctx_range=(0, 40), n_steps=2, hidden=hidden)
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain_catchup(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = [0, batch - 1] if batch > 1 else [0]
    orc, hi = oracle_for(cfg, w, inp, seqs)
    log(cfg.name, check_chain(cfg, out, orc, hi, seqs, catchup=True, inp=inp))
    dr.close()


def test_catchup_features_at_any_address():
    """Features that are not 16-byte aligned take the staged operand, and give
    what the route that reads them in place gives (both against the oracle)."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_catchup_unaligned", batch=2, n_new=(50, 70), n_steps=2)
    dr, w, inp = gpu_setup(cfg)
    orc, hi = oracle_for(cfg, w, inp, [0, 1])
    flat = torch.zeros(inp.new_features.numel() + 8, dtype=torch.bfloat16, device="cuda")
    for shift in (0, 1, 4):
        view = flat[shift:shift + inp.new_features.numel()].view_as(inp.new_features)
        view.copy_(inp.new_features)
        assert (view.data_ptr() % 16 == 0) == (shift == 0)
        x = type(inp)(**{**inp.__dict__, "new_features": view})
        out = dr.chain_catchup(x, logits=True, hidden=True)
        torch.cuda.synchronize()
        assert dr.device_status() == 0
        check_chain(cfg, out, orc, hi, [0, 1], catchup=True, inp=inp)
    dr.close()


def test_long_catchup_flags_bad_tokens():
    cfg = SMALL_BF16_CHAIN.with_(name="small_catchup_badtok", batch=1, n_new=(80, 80), n_steps=1)
    dr, w, inp = gpu_setup(cfg)
    good = inp.new_tokens.clone()
    inp.new_tokens[7] = cfg.vocab
    dr.chain_catchup(inp)
    assert dr.device_status() == -1
    inp.new_tokens.copy_(good)
    dr.chain_catchup(inp)
    assert dr.device_status() == 0
    dr.close()


def test_long_catchup_flags_malformed_offsets():
    """A sequence without rows in a front of more than 64: its last row reads as
    zeros, the flag is the offsets', and a later call is clean."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_catchup_badoff", batch=3, n_new=(30, 30), n_steps=1)
    dr, w, inp = gpu_setup(cfg)
    good = inp.new_offsets.clone()
    inp.new_offsets = torch.tensor([0, 50, 50, 90], dtype=torch.int32, device="cuda")
    dr.chain_catchup(inp)
    assert dr.device_status() == -1
    inp.new_offsets = good
    out = dr.chain_catchup(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    orc, hi = oracle_for(cfg, w, inp, [0, 2])
    check_chain(cfg, out, orc, hi, [0, 2], catchup=True, inp=inp)
    dr.close()


def test_long_front_sums_stay_short():
    """2048 accepted rows at hidden 2304: one K slice of 384 k-blocks of the
    fusion FC.  All terms positive, so the running sum grows steadily and each
    addition rounds at about the sum's size so far: 2^-24 / sqrt(3) / 1.44 of
    it (rms).  One chain of 384 additions is off by sqrt(384 / 3) = 11.3 of
    these (2.7e-7); sums of at most 32, then 12 of those, by sqrt(32 / 3 / 12)
    and sqrt(12 / 3) = 2.2 (5e-8, and a few more roundings after the sum).  The
    line lies at 5.5.  With W_o, W_down and E zero the step's hidden row is the
    FC's output."""
    H, F, T = 2304, 12288, 2048
    cfg = SMALL_BF16_CHAIN.with_(name="small_long_sum", hidden=H, feat_width=F, batch=1, n_new=(T, T), n_steps=1,
                                 n_sets=1, f_map=(0,), ctx_range=(0, 0))
    w, inp = make_weights(cfg, "cuda"), make_inputs(cfg, "cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    ps = w.sets[0]
    ps.w_fc.copy_(torch.rand(ps.w_fc.shape, generator=g, device="cuda") + 0.5)
    inp.new_features.copy_(torch.rand(inp.new_features.shape, generator=g, device="cuda") + 0.5)
    for t in (ps.w_o, ps.w_down, w.embed):
        t.zero_()
    from paper_2602_01762_amd import Drafter
    dr = Drafter(cfg)
    dr.load(w)
    out = dr.chain_catchup(inp, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    want = ps.w_fc[:, H:].double().cpu().numpy() @ inp.new_features[-1].double().cpu().numpy()
    rel = out["hidden"][0, 0].double().cpu().numpy() / want - 1
    rms = float(np.sqrt(np.mean(rel ** 2)))
    log(cfg.name, rms)
    assert rms <= 5.5 * 2 ** -24 / 3 ** 0.5 / 1.44
    dr.close()


# k-blocks of the one slice of the front's fusion FC: at, below and past one and
# two running sums of 32, and fewer than the loads in flight
@pytest.mark.parametrize("kblocks", [1, 3, 31, 32, 33, 34, 64, 65])
def test_long_front_running_sum_edges(kblocks):
    """2048 accepted rows at hidden 2304, random values: the FC's output in the
    last row (W_o, W_down and E zero) against fp64.  The features are one exact
    plane, so the error is fp32 rounding: each of up to 34 additions, of the
    sum's size times 2^-24, over a sum of F terms of size sqrt(F)."""
    H, F, T = 2304, 32 * kblocks, 2048
    cfg = SMALL_BF16_CHAIN.with_(name="small_fold_%d" % kblocks, hidden=H, feat_width=F, batch=1, n_new=(T, T),
                                 n_steps=1, n_sets=1, f_map=(0,), ctx_range=(0, 0))
    from paper_2602_01762_amd import Drafter
    w, inp = make_weights(cfg, "cuda"), make_inputs(cfg, "cuda")
    ps = w.sets[0]
    for t in (ps.w_o, ps.w_down, w.embed):
        t.zero_()
    dr = Drafter(cfg)
    dr.load(w)
    out = dr.chain_catchup(inp, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    want = ps.w_fc[:, H:].double().cpu().numpy() @ inp.new_features[-1].double().cpu().numpy()
    err = out["hidden"][0, 0].double().cpu().numpy() - want
    assert np.max(np.abs(err)) <= 34 * 2 ** -24 * 0.02 * F ** 0.5 * 5     # 5 sigma of the largest of 2304
    dr.close()


# one slice of 15, 16, 17 and 33 k-blocks at 64 rows (running sums of 16)
@pytest.mark.parametrize("hidden", [480, 512, 544, 1056])
def test_chain_running_sum_edges(hidden):
    cfg = SMALL_BF16_CHAIN.with_(name="small_fold64_%d" % hidden, batch=40, hidden=hidden, ffn=16416, n_steps=2,
                                 ctx_range=(1, 60))
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    orc, hi = oracle_for(cfg, w, inp, [0, 39])
    log(cfg.name, check_chain(cfg, out, orc, hi, [0, 39], inp=inp))
    dr.close()


# trees x (nodes + 1) rows: one tree below the small kernels' limit, whole
# row tiles, one row past a tile, passes of whole trees; 1 node: 2 rows share
# a feature row; hidden 480: no embedding table; vocabulary 33040: more than
# 128 groups of 256 ids, the last ragged, where a head over more than 192 rows
# takes 256-row tiles
@pytest.mark.parametrize("batch,nodes,hidden,vocab", [
    (1, 60, 512, 5008), (2, 63, 512, 5008), (3, 42, 512, 5008), (1, 1, 512, 5008), (64, 1, 512, 5008),
    (9, 28, 512, 5008), (3, 42, 480, 5008), (3, 63, 512, 33040), (4, 48, 512, 33040), (4, 63, 512, 33040),
    (4, 60, 480, 33040)])
def test_score_rows_share_their_trees_features(batch, nodes, hidden, vocab):
    """Scoring with target features that are not zero: every row of a tree
    fuses its sequence's feature row."""
    from oracle import Oracle
    from paper_2602_01762_amd import Drafter
    cfg = scoring_target(SMALL_BF16_CHAIN.with_(
        name="small_score_%dx%d" % (batch, nodes), batch=batch, tree_nodes=nodes, tree_width=1,
        hidden=hidden, vocab=vocab, ctx_range=(3, 90)))
    w, inp = make_weights(cfg, "cuda"), make_inputs(cfg, "cuda")
    dr = Drafter(cfg)
    dr.load(w)
    rng = np.random.default_rng(batch * 100 + nodes)
    depth = np.ones((batch, nodes), np.int32)
    mask = np.zeros((batch, nodes), np.uint64)
    for b in range(batch):
        for j in range(nodes):
            p = int(rng.integers(-1, j)) if j else -1
            depth[b, j] = 1 if p < 0 else depth[b, p] + 1
            mask[b, j] = (np.uint64(0) if p < 0 else mask[b, p]) | (np.uint64(1) << np.uint64(j))
    toks = rng.integers(0, cfg.vocab, (batch, nodes)).astype(np.int32)
    dev = lambda x: torch.tensor(x, device="cuda")
    lg = dr.score_tree(inp, dev(toks), dev(depth), dev(mask.view(np.int64)))
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = sorted({0, batch // 2, batch - 1})
    ref = Oracle(cfg, host_weights(w)).score_tree(host_inputs(inp, cfg, seqs), toks, depth, mask, seqs)
    for b in seqs:
        assert np.max(np.abs(lg[b].cpu().numpy() - ref["logits"][b])) <= LOGIT_TOL["bf16"], b
    check_draft_kv(cfg, inp, ref["draft_kv"], seqs)
    dr.close()


# 33 rows or more take the tile kernel at 64 rows per workgroup, 32 the
# streaming kernels; 4 to 16 rows read the same fragments with lanes past the
# last row folded onto row 0
@pytest.mark.parametrize("batch", [2, 3, 16, 17, 32, 33, 47, 48, 64])
@pytest.mark.parametrize("kv_block", [16, 24])
def test_chain_row_counts(batch, kv_block):
    """Chains at the edges of the row tiles, with a KV block size that is a
    power of two and one that is not."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_rows_%d_%d" % (batch, kv_block), batch=batch, n_steps=2,
                                 ctx_range=(1, 90), kv_block_size=kv_block)
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = sorted({0, batch // 2, batch - 1})
    orc, hi = oracle_for(cfg, w, inp, seqs)
    log(cfg.name, check_chain(cfg, out, orc, hi, seqs, inp=inp))
    dr.close()


# 320 vocab tiles: 8 per wave up to 32 rows, 4 above; 322: 2 per wave
@pytest.mark.parametrize("batch,vocab", [(32, 5120), (33, 5120), (48, 5120), (64, 5120), (49, 5152)])
def test_chain_lm_head_tiles(batch, vocab):
    cfg = SMALL_BF16_CHAIN.with_(name="small_lm_%d_%d" % (batch, vocab), batch=batch, vocab=vocab, n_steps=2,
                                 ctx_range=(1, 90))
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = sorted({0, batch // 2, batch - 1})
    orc, hi = oracle_for(cfg, w, inp, seqs)
    log(cfg.name, check_chain(cfg, out, orc, hi, seqs, inp=inp))
    dr.close()


@pytest.mark.parametrize("batch", [33, 40, 64])
def test_chain_steps_without_prep_above_32_rows(batch):
    """Steps >= 2 whose fusion FC has at least a workgroup per row (hidden 2048:
    8 tile groups x 8 to 15 slices) resolve their tokens in that product, on
    the streaming kernel with the slices of the tile kernel's plan."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_direct_%d" % batch, batch=batch, hidden=2048, n_steps=3,
                                 ctx_range=(1, 60))
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = sorted({0, batch // 2, batch - 1})
    orc, hi = oracle_for(cfg, w, inp, seqs)
    log(cfg.name, check_chain(cfg, out, orc, hi, seqs, inp=inp))
    dr.close()


def test_chain_shared_reduction_of_eight_tiles():
    """Gate/up of 1600 tiles at 24 rows: 4 waves of 8 tiles x 2 row tiles,
    66.8 KB of LDS (the plan is checked by test_shared_reduction_fits_the_lds)."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_ffn12800_h1024", batch=24, hidden=1024, ffn=12800, n_steps=2,
                                 ctx_range=(1, 90))
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    seqs = [0, 11, 23]
    orc, hi = oracle_for(cfg, w, inp, seqs)
    log(cfg.name, check_chain(cfg, out, orc, hi, seqs, inp=inp))
    dr.close()


@pytest.mark.parametrize("head_dim,nq,nkv", [(32, 8, 2), (64, 4, 4), (128, 4, 1), (256, 2, 2)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attention_head_dims(head_dim, nq, nkv, dtype):
    """Every head width of the VALU and the matrix-core attention, contexts of
    less than a step and of several chunks; positions up to 5000 rotate."""
    cfg = SMALL_BF16_CHAIN.with_(name="small_d%d_%s" % (head_dim, dtype), head_dim=head_dim, n_q_heads=nq,
                                 n_kv_heads=nkv, dtype=dtype, batch=2, n_steps=2, ctx_range=(5, 5000))
    dr, w, inp = gpu_setup(cfg)
    out = dr.chain(inp, logits=True, hidden=True)
    torch.cuda.synchronize()
    assert dr.device_status() == 0
    orc, hi = oracle_for(cfg, w, inp, [0, 1])
    log(cfg.name, check_chain(cfg, out, orc, hi, [0, 1], inp=inp))
    dr.close()
