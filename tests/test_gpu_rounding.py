"""Roundings that later results hang on: a panel element that changes by its last bit moves cache entries by a bf16 step."""
import numpy as np
import pytest
import torch

from paper_2405_04304_amd import binding as B
from workloads import synth as W

from test_gpu_parity import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,chunk", [(1024, 1024), (2048, 1024), (4096, 4096), (5120, 4096), (8192, 4096)])
def test_embedding_norm_panels_bit_by_bit(d, chunk):
    """The panels of gain * h of the first norm: lo is what hi leaves of the exact product in a row's first chunk of columns (four per
    thread) and of the product rounded to fp32 beyond it.  Query projection = identity, one token at position 0, so query
    row = (hi + lo) / rms in fp32; h is a multiple of 1 / 16, so the sum of squares is exact in any order."""
    rng = np.random.default_rng(d)
    shape = W.ModelShape("B", 1, d, d // 64, 64, 1, 64, 64)
    h = (rng.integers(1, 16, d) / 16.0 * rng.choice([-1.0, 1.0], d)).astype(np.float32)
    gain = (1.0 + 0.1 * rng.standard_normal(d)).astype(np.float32)
    bf16 = torch.bfloat16
    zeros = lambda *n: torch.zeros(*n, dtype=bf16)  # noqa: E731
    qkv = zeros(d + 128, d)
    qkv[:d] = torch.eye(d, dtype=bf16)
    emb = zeros(64, d)
    emb[3] = torch.from_numpy(h).to(bf16)
    w = {"tok_emb": emb, "wlm": zeros(64, d), "normf_g": torch.ones(d), "l0.norm1_g": torch.from_numpy(gain), "l0.norm2_g": torch.ones(d),
         "l0.wqkv": qkv, "l0.wo": zeros(d, d), "l0.wg": zeros(64, d), "l0.wu": zeros(64, d), "l0.wd": zeros(d, 64)}
    gm = B.DiscoModel(shape, w, dev())
    gkv, ws = B.DiscoKV(gm, 16, 16), gm.workspace(16, 16)
    am = torch.zeros(16, dtype=torch.int32, device=dev())
    B.disco_verify(gm, gkv, torch.tensor([3], dtype=torch.int32, device=dev()), 1, am, None, ws)
    torch.cuda.synchronize()
    first = (64 * d + 255) // 256 * 256                # query rows, behind the 16 residual rows
    got = ws.buf[first:first + 4 * d].view(torch.float32).cpu().numpy()
    exact = h.astype(np.float64) * gain                # 4 x 24 bits
    rounded = exact.astype(np.float32)
    cut = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(bf16).to(torch.float32).numpy()  # noqa: E731
    hi = cut(rounded)
    lo = np.where(np.arange(d) < chunk, cut((exact - hi).astype(np.float32)), cut(rounded - hi))
    assert (cut((exact - hi).astype(np.float32)) != cut(rounded - hi)).any()
    rstd = np.float32(1.0) / np.sqrt(np.float32((h.astype(np.float64) ** 2).sum()) / np.float32(d) + np.float32(shape.rms_eps))
    want = (hi + lo) * rstd
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, (bad.size, bad[:8], got[bad[:4]], want[bad[:4]])


@pytest.mark.parametrize("vocab", [4096, 32000])
@pytest.mark.parametrize("force", [None, 7])
def test_features_of_logits_that_are_not_numbers(vocab, force):
    """A NaN logit shows in every feature, also where its 256 neighbours (a wavefront's share) weigh nothing beside the largest logit or
    are NaN themselves; a wavefront's share of -inf weighs nothing.  One workgroup and many agree."""
    from test_gpu_parity import _run_classify
    clf = W.make_classifier(100)
    base = torch.randn(vocab, generator=torch.Generator().manual_seed(1))
    for first, width, value, around in ((1100, 1, float("nan"), -300.0), (1024, 256, float("nan"), None),
                                        (1024, 256, -float("inf"), None), (2048, 1024, -float("inf"), None)):
        x = base.clone()
        if around is not None:
            x[1024:1280] = around
        x[first:first + width] = value
        one, many = (_run_classify(x, clf, 3, 0.5, force, multi=m)[0] for m in (False, True))
        if value != value:
            assert all(f != f for f in list(one.feats)[:11]) and all(f != f for f in list(many.feats)[:11]), (first, list(many.feats))
        else:
            assert torch.allclose(torch.tensor(list(many.feats)), torch.tensor(list(one.feats)), rtol=1e-5, atol=1e-7)
        assert one.token == many.token
