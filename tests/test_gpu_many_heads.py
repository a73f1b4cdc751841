"""Head counts beyond 16 bits: nothing on the way to the attention may cut them."""
import pytest
import torch

from paper_2405_04304_amd import binding as B
from workloads import synth as W

from test_gpu_parity import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nh, nkv", [(65536, 1), (32768, 32768), (65544, 8)])
def test_copies_of_eight_heads_give_what_eight_heads_give(nh, nkv):
    """A model whose heads are copies of eight heads, each copy's output projection scaled by one over the copies' number, is that model of
    eight heads up to the order of the sums (64 x as many products as a 13B row: 2e-4 of the row's scale, the bar between launch structures)."""
    small = W.ModelShape("B", 1, 64, 8, 64, 1 if nkv == 1 else 8, 64, 64)
    w = W.make_weights(small, 4, "bf16", sigma=0.2)
    w = {k: v.to(dev()) for k, v in w.items()}
    copies = nh // 8
    big = W.ModelShape("B", 1, 64, nh, 64, nkv, 64, 64)
    dq = 8 * 64
    qkv = w["l0.wqkv"]
    q, kv = qkv[:dq], qkv[dq:].view(2, -1, 64)
    if nkv == 8:                                       # heads of a group are neighbours: copies of one head each
        q = q.view(8, 1, 64 * 64).expand(8, copies, 64 * 64).reshape(-1, 64)
        wo = (w["l0.wo"].float() / copies).to(torch.bfloat16).view(64, 8, 1, 64).expand(64, 8, copies, 64).reshape(64, -1)
    else:
        q = q.repeat(copies, 1)
        kv = kv.repeat(1, copies if nkv > 1 else 1, 1)
        wo = (w["l0.wo"].float() / copies).to(torch.bfloat16).repeat(1, copies)
    wb = dict(w)
    wb["l0.wqkv"], wb["l0.wo"] = torch.cat([q, kv.reshape(-1, 64)]), wo
    ws_ = dict(w)
    ws_["l0.wo"] = ((w["l0.wo"].float() / copies).to(torch.bfloat16).double() * copies).to(torch.bfloat16)
    ctx, got = 40, []
    for shape, weights in ((small, ws_), (big, wb)):
        gm = B.DiscoModel(shape, weights, dev())
        fill = W.make_kv_fill(small, ctx, 3).to(dev())
        if shape.n_kv_heads > small.n_kv_heads:
            fill = fill.repeat(1, 1, 1, copies, 1)
        gkv, ws, pws = B.DiscoKV(gm, 96, 16), gm.workspace(16, 96), gm.prefill_workspace(20, 96)
        out = []
        for M in (1, 12):
            gkv.fill(fill.contiguous())
            lg, am = torch.empty(M, 64, device=dev()), torch.zeros(16, dtype=torch.int32, device=dev())
            B.disco_verify(gm, gkv, W.make_tokens(7, M, 64).to(dev()), M, am, lg, ws)
            out.append(lg)
        gkv.fill(fill.contiguous())
        last = torch.empty(64, device=dev())
        B.disco_prefill(gm, gkv, W.make_tokens(8, 20, 64).to(dev()), 20, last, pws)
        torch.cuda.synchronize()
        got.append(out + [last])
        del gm, gkv, ws, pws
    for a, b in zip(*got):
        assert bool(torch.isfinite(b).all()) and float((a - b).abs().max()) <= 2e-4 * float(a.abs().max())
