"""All layers of a narrow model's forward over one or two tokens in one launch, against a launch per phase (mode 2) and the oracle.  Models whose
context is dealt the same way in both must agree bit by bit, logits and cache (the launch forms every sum in the same order); models with
a K / V head per query head have another deal in mode 2, so they agree to fp32 summation order there."""
import pytest
import torch

from paper_2405_04304_amd import binding as B
from workloads import synth as W

from test_gpu_fused_qkv_attn import _verify
from test_gpu_parity import check_argmax, check_logits, dev, setup_pair

pytestmark = pytest.mark.gpu

# family, layers, d_model, heads, head width, K / V heads, d_ff, vocab
SHAPES = {
    "one K / V head, 12 query heads": W.ModelShape("A", 3, 768, 12, 64, 1, 3072, 512),
    "3 K / V heads of 4, RMSNorm": W.ModelShape("B", 2, 768, 12, 64, 3, 2048, 512),
    "16 query heads on one, more columns than a product has with two tokens": W.ModelShape("A", 1, 512, 16, 64, 1, 768, 512),
    "heads of their own, LayerNorm": W.ModelShape("A", 2, 192, 3, 64, 3, 96, 320),
    "widest rows": W.ModelShape("A", 1, 1024, 8, 64, 2, 1024, 512),
    "narrowest": W.ModelShape("A", 2, 64, 1, 64, 1, 64, 64),
    "d_q above d_model, ragged K ranges": W.ModelShape("B", 2, 128, 8, 64, 2, 1760, 320),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_one_launch_and_a_launch_per_phase_agree_bit_by_bit(name):
    """Contexts at the edges of the deal (256, 768, 1536 positions), of a wavefront's 32 positions and of pages."""
    shape = SHAPES[name]
    gm = B.DiscoModel(shape, W.make_weights(shape, 90, "bf16", sigma=0.05), dev())
    for i, ctx in enumerate((0, 1, 31, 32, 254, 255, 256, 300, 766, 768, 1100, 1535, 1536, 3071)):
        page_tokens, capacity = (16, 4, 64, 8)[i % 4], ctx + 16
        n_pages = -(-capacity // page_tokens)
        order = torch.randperm(n_pages, generator=torch.Generator().manual_seed(i)).tolist() if i % 3 else None
        fill = W.make_kv_fill(shape, ctx, 3).to(dev()) if ctx else None
        for M in (1, 2):
            assert B.disco_layers_plan(gm.handle, M, ctx, page_tokens)["one_launch"]
            out, blk = [], W.make_tokens(80 + M, M, shape.vocab).tolist()
            for mode in (0, 2):
                gkv, ws = B.DiscoKV(gm, capacity, page_tokens, order), gm.workspace(16, capacity)
                if fill is not None:
                    gkv.fill(fill)
                lg, am = _verify(gm, gkv, ws, blk, mode)
                B.disco_kv_rollback(gkv, ctx)
                if ctx:                                # a second pass over the same workspace and cache
                    again, _ = _verify(gm, gkv, ws, blk, mode)
                    assert torch.equal(lg, again), (ctx, M, mode)
                # the block's entries are read back by a later token
                tail = _verify(gm, gkv, ws, blk[:1], mode)[0]
                out.append((lg, am, tail))
            assert bool(torch.isfinite(out[0][0]).all())
            assert torch.equal(out[0][0], out[1][0]) and out[0][1] == out[1][1] and torch.equal(out[0][2], out[1][2]), (ctx, M, page_tokens)


@pytest.mark.parametrize("ctx, page_tokens", [(0, 16), (100, 8), (255, 64), (523, 16), (1300, 32), (2475, 16)])
def test_heads_with_keys_of_their_own_against_the_oracle(ctx, page_tokens):
    shape = W.scaled_shape(W.CFG1_DRAFT, vocab=4096)
    om, gm, okv, gkv, ws = setup_pair(shape, 31, kv_ctx=ctx, capacity=ctx + 32, page_tokens=page_tokens, permute=True, sigma=0.04)
    for M in (1, 2):
        assert B.disco_layers_plan(gm.handle, M, ctx, page_tokens)["one_launch"]
        blk = W.make_tokens(60 + M, M, shape.vocab).tolist()
        ref = om.forward(blk, okv)
        okv.rollback(ctx)
        lg, am = _verify(gm, gkv, ws, blk, 0)
        B.disco_kv_rollback(gkv, ctx)
        lg2, _ = _verify(gm, gkv, ws, blk, 2)
        B.disco_kv_rollback(gkv, ctx)
        check_logits(lg, ref, f"one launch, ctx {ctx}, M {M}")
        check_argmax(am, ref, f"one launch, ctx {ctx}")
        assert float((lg - lg2).abs().max()) <= 2e-4 * float(lg2.abs().max())


@pytest.mark.parametrize("ctx, parts", [(1300, (3, 3)), (1700, (4, 4)), (2400, (5, 5)), (3071, (5, 4))])
def test_the_context_of_many_heads_over_more_workgroups(ctx, parts):
    """Sixteen heads of their own: as many workgroups a head as ranges of 512 positions, or pairs of shorter ranges; the same bits."""
    shape = W.ModelShape("A", 2, 128, 16, 64, 16, 512, 512)
    gm = B.DiscoModel(shape, W.make_weights(shape, 90, "bf16", sigma=0.05), dev())
    fill = W.make_kv_fill(shape, ctx, 3).to(dev())
    for M in (1, 2):
        plan = B.disco_layers_plan(gm.handle, M, ctx, 16)
        assert plan["one_launch"] and plan["groups"] == 16 and plan["parts"] == parts[M - 1]
        blk, out = W.make_tokens(80 + M, M, shape.vocab).tolist(), []
        for mode in (0, 2):
            gkv, ws = B.DiscoKV(gm, ctx + 32, 16), gm.workspace(16, ctx + 32)
            gkv.fill(fill)
            out.append(_verify(gm, gkv, ws, blk, mode)[0])
        assert bool(torch.isfinite(out[0]).all()) and torch.equal(out[0], out[1]), M


def test_captured_forward_replays():
    """Replays of a captured forward, which holds a launch per phase, between eager ones with all layers in one launch, on one workspace: the same bits."""
    d = dev()
    shape = SHAPES["one K / V head, 12 query heads"]
    gm = B.DiscoModel(shape, W.make_weights(shape, 90, "bf16", sigma=0.05), d)
    gkv, ws = B.DiscoKV(gm, 332, 16), gm.workspace(16, 332)
    gkv.fill(W.make_kv_fill(shape, 300, 3).to(d))
    toks = [torch.tensor([7 + 3 * i], dtype=torch.int32, device=d) for i in range(4)]
    lg, tok = torch.empty(shape.vocab, device=d), toks[0].clone()
    want = []
    for t in toks:
        B.disco_draft_step(gm, gkv, t, 1, lg, ws)
        B.disco_kv_rollback(gkv, 300)
        want.append(lg.clone())
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        B.disco_draft_step(gm, gkv, tok, 1, lg, ws)
    B.disco_kv_rollback(gkv, 300)
    for rep in range(3):
        for t, w in zip(toks, want):
            tok.copy_(t)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(lg, w), rep
        B.disco_draft_step(gm, gkv, toks[rep], 1, lg, ws)
        B.disco_kv_rollback(gkv, 300)
        assert torch.equal(lg, want[rep])


def test_a_wait_that_gives_up_is_reported():
    """The limit forced to 'give up at once' from the host: every wavefront still runs to its end, and every result channel says so."""
    shape = SHAPES["3 K / V heads of 4, RMSNorm"]
    gm = B.DiscoModel(shape, W.make_weights(shape, 90, "bf16", sigma=0.05), dev())
    gkv, ws = B.DiscoKV(gm, 932, 16), gm.workspace(16, 932)
    gkv.fill(W.make_kv_fill(shape, 900, 3).to(dev()))
    blk = W.make_tokens(3, 2, shape.vocab).tolist()
    want, want_am = _verify(gm, gkv, ws, blk, 0)
    B.disco_kv_rollback(gkv, 900)
    prev = B.disco_set_wait_limit(-1)
    try:
        lg, am = _verify(gm, gkv, ws, blk, 0)
    finally:
        B.disco_set_wait_limit(prev)
    B.disco_kv_rollback(gkv, 900)
    assert am == [-1, -1] and bool(torch.isnan(lg).all())
    B.lib().disco_workspace_init(gm.handle, ws.buf.data_ptr(), ws.nbytes, 16, 932, B._stream())
    lg, am = _verify(gm, gkv, ws, blk, 0)
    assert am == want_am and torch.equal(lg, want)
