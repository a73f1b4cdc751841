"""The many-workgroup classify (records handed over by polling) against the one-workgroup form, which sorts by rounds: edges of the slices of 1024
logits and of the wavefronts' 256, rows with fewer than ten numbers, rows whose candidates do not fit a list (many equal logits), and a wait that gives up."""
import pytest
import torch

from paper_2405_04304_amd import binding as B
from paper_2405_04304_amd.engine import SpecEngine
from workloads import synth as W

from test_gpu_parity import dev

pytestmark = pytest.mark.gpu


def _row(kind, vocab, g):
    x = torch.randn(vocab, generator=g)
    if kind == "equal":
        x = torch.full((vocab,), 0.25)
    elif kind == "few values":
        x = torch.randint(0, 3, (vocab,), generator=g).float()
    elif kind == "seven numbers":
        y = torch.full((vocab,), float("-inf"))
        at = torch.randperm(vocab, generator=g)[:7]
        y[at] = x[at]
        x = y
    elif kind == "one slice":                            # all of the ten largest, and equal ones, in the last slice
        x[-200:-150] = 9.0
    elif kind == "zeros and signs":
        x = torch.where(x > 0, 0.0, -0.0)
    return x


def _classify(clf, x, force, scratch):
    d = dev()
    rec = B.struct_tensor(B.ClfOut, 1, d)
    lg = x.to(d).contiguous()
    f = torch.tensor([force], dtype=torch.int32, device=d) if force is not None else None
    B.disco_classify(clf, lg, x.numel(), 3.0, 0.5, False, rec, force_token=f, scratch=scratch)
    torch.cuda.synchronize()
    return B.read_struct(B.ClfOut, rec, 0), lg.cpu()


@pytest.mark.parametrize("kind", ["normal", "equal", "few values", "seven numbers", "one slice", "zeros and signs"])
def test_records_against_one_workgroup(kind):
    g = torch.Generator().manual_seed(5)
    scratch = B.classify_scratch(dev())
    clf = B.DiscoClf(W.make_classifier(100), dev())
    for vocab in (4096, 4097, 5119, 5120, 5376, 32000, 49152, 65535, 65536):
        x = _row(kind, vocab, g)
        for force in (None, int(torch.argmax(x)), vocab - 1):
            (a, la), (b, lb) = _classify(clf, x, force, scratch), _classify(clf, x, force, None)
            assert a.token == b.token and a.halt == b.halt and a.executed == b.executed == 1, (vocab, force)
            # the same logits are selected; sums in another order: a few units in the last place of the probabilities, of the entropy's terms (< 12) absolutely
            assert torch.allclose(torch.tensor(list(a.feats)), torch.tensor(list(b.feats)), rtol=2e-6, atol=5e-6), (vocab, force)
            assert abs(a.score - b.score) < 1e-5 and torch.equal(la, lb)
    assert int(scratch.view(torch.int32).abs().sum()) == 0           # every launch leaves its scratch empty


def test_a_wait_that_gives_up_is_reported():
    scratch = B.classify_scratch(dev())
    clf = B.DiscoClf(W.make_classifier(100), dev())
    x = _row("normal", 32000, torch.Generator().manual_seed(6))
    want = _classify(clf, x, None, scratch)[0]
    prev = B.disco_set_wait_limit(-1)
    try:
        got = _classify(clf, x, None, scratch)[0]
    finally:
        B.disco_set_wait_limit(prev)
    assert got.token == -1 and got.halt == 1 and got.score != got.score
    B._check(B.lib().disco_classify_scratch_init(scratch.data_ptr(), B._stream()))
    again = _classify(clf, x, None, scratch)[0]
    assert list(again.feats) == list(want.feats) and again.token == want.token and again.score == want.score


@pytest.mark.parametrize("arrived", ["ten largest", "statistics"])
def test_either_polling_wavefront_may_give_up_alone(arrived):
    """Two wavefronts poll different words of the records.  With one part in place beforehand and a limit of one poll, one of them succeeds and the other
    runs out: the call reports the failure."""
    scratch = B.classify_scratch(dev())
    clf = B.DiscoClf(W.make_classifier(100), dev())
    x = _row("normal", 32000, torch.Generator().manual_seed(6))
    recs = scratch.view(torch.int32)[64:].view(64, 16)
    (recs[:, 4:] if arrived == "ten largest" else recs[:, :4]).fill_(0x7F000000)
    prev = B.disco_set_wait_limit(0)
    try:
        got = _classify(clf, x, None, scratch)[0]
    finally:
        B.disco_set_wait_limit(prev)
    assert got.token == -1 and got.halt == 1 and got.score != got.score and got.executed == 1


def test_a_give_up_stays_on_its_scratch_until_that_is_initialised():
    """A workgroup that is late stores its record behind the give-up: no later call may take that for a record of its own row."""
    scratch = B.classify_scratch(dev())
    clf = B.DiscoClf(W.make_classifier(100), dev())
    g = torch.Generator().manual_seed(7)
    x, y = _row("normal", 32000, g), _row("normal", 32000, g)
    want = _classify(clf, y, None, scratch)[0]
    prev = B.disco_set_wait_limit(-1)
    try:
        assert _classify(clf, x, None, scratch)[0].token == -1
    finally:
        B.disco_set_wait_limit(prev)
    for _ in range(3):
        got = _classify(clf, y, None, scratch)[0]
        assert got.token == -1 and got.halt == 1 and got.score != got.score and got.executed == 1
    B._check(B.lib().disco_classify_scratch_init(scratch.data_ptr(), B._stream()))
    for _ in range(2):
        got = _classify(clf, y, None, scratch)[0]
        assert got.token == want.token and list(got.feats) == list(want.feats) and got.score == want.score


def test_a_give_up_on_the_array_of_the_library_ends_with_its_call():
    d, clf = dev(), B.DiscoClf(W.make_classifier(100), dev())
    g = torch.Generator().manual_seed(8)
    x, y = _row("normal", 32000, g).to(d), _row("normal", 32000, g).to(d)
    rec = B.struct_tensor(B.ClfOut, 1, d)

    def call(t):
        B.disco_classify_static(clf, t, 32000, 3.0, 0.5, 0, rec)
        torch.cuda.synchronize()
        return B.read_struct(B.ClfOut, rec, 0)

    want = call(y)
    prev = B.disco_set_wait_limit(-1)
    try:
        assert call(x).token == -1
    finally:
        B.disco_set_wait_limit(prev)
    got = call(y)
    assert got.token == want.token and list(got.feats) == list(want.feats) and got.score == want.score


def _draft_loop(gm, clf, ws, ctx, tau=0.0, ppl=0.0):
    d = dev()
    kv = B.DiscoKV(gm, ctx + 32, 16)
    B.disco_kv_rollback(kv, 0)
    steps, lo_d, lo_h = B.struct_tensor(B.ClfOut, 16, d), B.struct_tensor(B.LoopOut, 1, d), B.struct_tensor(B.LoopOut, 1, pinned=True)
    tok, lg = torch.tensor([5], dtype=torch.int32, device=d), torch.empty(gm.shape.vocab, dtype=torch.float32, device=d)
    B.disco_draft_loop_ex(gm, kv, clf, tok, 1, 3, 0, 1.0, tau, lg, steps, lo_d, lo_h, ws, ppl_threshold=ppl)
    torch.cuda.synchronize()
    lo = B.LoopOut.from_buffer_copy(lo_h.numpy().tobytes())
    return lo.sl, list(lo.block[:4]), bool(torch.isfinite(lg).all())


def test_a_give_up_inside_a_draft_loop_is_reported():
    """A model whose forward waits nowhere (68 heads of their own, at most 256 positions: a launch per phase), so the features' launch is the only wait
    of its draft loop: the loop reports -1 and an iteration DISCO_EHIP until the workspace is initialised, as for every other wait."""
    d = dev()
    shape = W.ModelShape("B", 1, 64, 68, 64, 68, 64, 4096)
    gm, clf = B.DiscoModel(shape, W.make_weights(shape, 9, "bf16", sigma=0.05), d), B.DiscoClf(W.make_classifier(100), d)
    assert B.disco_qkv_attn_plan(gm.handle, 1, 40)["form"] == "separate" and not B.disco_layers_plan(gm.handle, 1, 40, 16)["one_launch"]
    ws = gm.workspace(16, 96)
    for kind in ("classifier", "perplexity"):
        args = {"tau": 0.0} if kind == "classifier" else {"ppl": 1e30}
        c = clf if kind == "classifier" else None
        want = _draft_loop(gm, c, ws, 40, **args)
        assert want[0] == 3 and want[2]
        prev = B.disco_set_wait_limit(-1)
        try:
            assert _draft_loop(gm, c, ws, 40, **args)[0] == -1
        finally:
            B.disco_set_wait_limit(prev)
        assert _draft_loop(gm, c, ws, 40, **args)[0] == -1                    # the workspace stays marked
        B._check(B.lib().disco_workspace_init(gm.handle, ws.buf.data_ptr(), ws.nbytes, 16, 96, B._stream()))
        assert _draft_loop(gm, c, ws, 40, **args) == want
    eng = SpecEngine(gm, gm, clf, max_ctx=96)
    prompt, pol = list(range(5, 25)), {"mode": "disco", "tau": 0.0, "sl_max": 3, "pos_mode": "block"}
    text = eng.generate(prompt, 8, pol)["tokens"]
    for extra in ({}, {"mode": "oracle", "reference": text}):
        eng.reset()
        eng.prefill(prompt[:-1])
        prev = B.disco_set_wait_limit(-1)
        try:
            with pytest.raises(B.DiscoError) as e:
                eng.generate(prompt, 8, dict(pol, **extra), do_prefill=False)
            assert e.value.code == B.EHIP
        finally:
            B.disco_set_wait_limit(prev)
        B._check(B.lib().disco_workspace_init(gm.handle, eng.ws_d.buf.data_ptr(), eng.ws_d.nbytes, 16, 96, B._stream()))
        assert eng.generate(prompt, 8, dict(pol, **extra))["tokens"] == text


@pytest.mark.parametrize("vocab", [4096, 5119, 32000, 65536])
def test_launch_mode_2_waits_nowhere(vocab):
    """In launch mode 2 the last workgroup to arrive merges: the same bits, with every bounded wait forced to give up at once."""
    scratch, clf = B.classify_scratch(dev()), B.DiscoClf(W.make_classifier(100), dev())
    x = _row("normal", vocab, torch.Generator().manual_seed(9))
    for force in (None, 17):
        want, wl = _classify(clf, x, force, scratch)
        prev_mode, prev = B.disco_set_launch_mode(2), B.disco_set_wait_limit(-1)
        try:
            got = [_classify(clf, x, force, scratch) for _ in range(2)]
        finally:
            B.disco_set_wait_limit(prev)
            B.disco_set_launch_mode(prev_mode)
        for r, l in got:
            assert r.token == want.token and list(r.feats) == list(want.feats) and r.score == want.score and r.halt == want.halt and torch.equal(l, wl)
        again = _classify(clf, x, force, scratch)[0]
        assert again.token == want.token and list(again.feats) == list(want.feats)
    assert int(scratch.view(torch.int32).abs().sum()) == 0
    shape = W.ModelShape("A", 2, 256, 4, 64, 4, 512, 4096)
    gm = B.DiscoModel(shape, W.make_weights(shape, 9, "bf16", sigma=0.05), dev())
    ws = gm.workspace(16, 96)
    prev_mode = B.disco_set_launch_mode(2)
    try:
        want = _draft_loop(gm, clf, ws, 40)
        prev = B.disco_set_wait_limit(-1)
        try:
            assert _draft_loop(gm, clf, ws, 40) == want and want[0] == 3
        finally:
            B.disco_set_wait_limit(prev)
    finally:
        B.disco_set_launch_mode(prev_mode)


def test_rows_with_logits_that_are_not_numbers():
    """A NaN among the logits, or infinities of one sign: token, halt and which features are numbers as the one-workgroup form has them."""
    scratch, clf = B.classify_scratch(dev()), B.DiscoClf(W.make_classifier(100), dev())
    g = torch.Generator().manual_seed(10)

    def num(r):
        return [f == f for f in list(r.feats) + [r.score]]

    for vocab in (4096, 32000, 65535):
        for kind in ("one", "last", "many", "all", "sign", "+inf", "-inf"):
            x = _row("normal", vocab, g)
            if kind in ("one", "last", "sign"):
                x[vocab - 1 if kind == "last" else 700] = float("nan")
                if kind == "sign":
                    x.view(torch.int32)[700] = -1                 # every bit set
            elif kind == "many":
                x[::7] = float("nan")
            elif kind == "all":
                x[:] = float("nan")
            elif kind == "+inf":
                x[123] = float("inf")
            else:
                x[:] = float("-inf")
            (a, _), (b, _) = _classify(clf, x, None, scratch), _classify(clf, x, None, None)
            if kind == "all":                                     # no arg-max: no token of the vocabulary, and an entropy that is no number
                assert min(a.token, b.token) >= vocab and a.feats[10] != a.feats[10] and b.feats[10] != b.feats[10] and a.halt == b.halt, vocab
            else:
                assert a.token == b.token and a.halt == b.halt and num(a) == num(b), (vocab, kind)
    assert int(scratch.view(torch.int32).abs().sum()) == 0
