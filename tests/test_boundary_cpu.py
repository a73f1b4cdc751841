"""The C boundary without a GPU: the library loads, exports every declared symbol, and rejects bad
arguments on the host before any launch (fake device addresses are never dereferenced)."""
import ctypes as C
import os
import re

import pytest

import paper_2405_04304_amd as D
from paper_2405_04304_amd import binding as B
from workloads import synth as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x7F0000000000  # 256-byte aligned address that is never touched


def _declared():
    names = set()
    for h in sorted(os.listdir(os.path.join(ROOT, "include"))):
        if h.endswith(".h"):
            names |= set(re.findall(r"\b(disco_[a-z_]+)\s*\(", open(os.path.join(ROOT, "include", h)).read()))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    lib = B.lib()
    names = _declared()
    assert set(names) == set(B.EXPORTS)
    for n in names:
        assert hasattr(lib, n), n


def _model(family=1, **over):
    d = dict(family=family, n_layers=2, d_model=64, n_heads=2, d_head=64, n_kv_heads=2, d_ff=128,
             vocab=256, max_pos=64, norm_eps=1e-5, rope_base=10000.0)
    d.update(over)
    desc = B.ModelDesc(*[d[k] for k in ("family", "n_layers", "d_model", "n_heads", "d_head", "n_kv_heads",
                                        "d_ff", "vocab", "max_pos", "norm_eps", "rope_base")])
    layers = (B.LayerWeights * d["n_layers"])()
    for L in layers:
        for f, _ in B.LayerWeights._fields_:
            setattr(L, f, FAKE)
    mw = B.ModelWeights(FAKE, d["d_model"], FAKE, layers, FAKE, FAKE, FAKE)
    h = C.c_void_p()
    rc = B.lib().disco_model_create(C.byref(desc), C.byref(mw), C.byref(h))
    return rc, h


def test_model_create_validation():
    rc, h = _model()
    assert rc == 0 and h.value
    B.lib().disco_model_destroy(h)
    assert _model(family=7)[0] == B.EINVAL
    assert _model(d_head=48)[0] == B.EINVAL
    assert _model(d_model=65)[0] == B.EINVAL
    assert _model(n_heads=3, n_kv_heads=2)[0] == B.EINVAL
    assert _model(vocab=250)[0] == B.EINVAL
    assert "vocab" in B.last_error() or "multiples" in B.last_error()


def _kv(model, capacity=40, page=16):
    nbytes = B.lib().disco_kv_bytes(model, capacity, page)
    h = C.c_void_p()
    rc = B.lib().disco_kv_create(model, FAKE, nbytes, capacity, page, None, C.byref(h))
    return rc, h, nbytes


def test_kv_and_rollback_host_logic():
    rc, m = _model()
    assert rc == 0
    lib = B.lib()
    rc, kv, nbytes = _kv(m)
    assert rc == 0 and nbytes > 0
    # capacity rounds up to whole pages: 40 -> 48
    assert lib.disco_kv_len(kv) == 0 and lib.disco_kv_pages_in_use(kv) == 0
    assert lib.disco_kv_rollback(kv, 0) == 0               # no-op on an empty cache
    assert lib.disco_kv_rollback(kv, 1) == B.ESTATE
    assert lib.disco_kv_rollback(kv, -1) == B.ESTATE
    assert lib.disco_kv_rollback(None, 0) == B.EINVAL
    h = C.c_void_p()
    assert lib.disco_kv_create(m, FAKE, nbytes - 1, 40, 16, None, C.byref(h)) == B.ECAP
    assert lib.disco_kv_create(m, FAKE + 8, nbytes, 40, 16, None, C.byref(h)) == B.EINVAL
    bad = (C.c_int32 * 3)(0, 0, 2)
    assert lib.disco_kv_create(m, FAKE, nbytes, 40, 16, bad, C.byref(h)) == B.EINVAL
    lib.disco_kv_destroy(kv)
    lib.disco_model_destroy(m)


def test_forward_calls_reject_bad_arguments_before_any_launch():
    rc, m = _model()
    rc2, other = _model()
    lib = B.lib()
    rc, kv, _ = _kv(m)
    ws = lib.disco_workspace_bytes(m, 16, 48)
    assert ws > 0 and lib.disco_workspace_bytes(m, 17, 48) == 0
    # null pointers
    assert lib.disco_draft_step(m, kv, None, 1, FAKE, FAKE, ws, None, None) == B.EINVAL
    assert lib.disco_draft_step(m, kv, FAKE, 1, None, FAKE, ws, None, None) == B.EINVAL
    assert lib.disco_verify(m, kv, FAKE, 1, None, None, FAKE, ws, None) == B.EINVAL
    # block length outside [1, 16]
    assert lib.disco_verify(m, kv, FAKE, 0, FAKE, None, FAKE, ws, None) == B.ECAP
    assert lib.disco_verify(m, kv, FAKE, 17, FAKE, None, FAKE, ws, None) == B.ECAP
    assert lib.disco_draft_step(m, kv, FAKE, 0, FAKE, FAKE, ws, None, None) == B.ECAP
    # workspace too small / misaligned
    assert lib.disco_verify(m, kv, FAKE, 4, FAKE, None, FAKE, 1024, None) == B.EINVAL
    assert lib.disco_verify(m, kv, FAKE, 4, FAKE, None, FAKE + 4, ws, None) == B.EINVAL
    # KV handle of another model
    assert lib.disco_verify(other, kv, FAKE, 4, FAKE, None, FAKE, ws, None) == B.ESTATE
    # accept / classify / loop argument checks
    assert lib.disco_accept(FAKE, FAKE, 0, None, FAKE, None, None) == B.ECAP
    assert lib.disco_accept(None, FAKE, 4, None, FAKE, None, None) == B.EINVAL
    assert lib.disco_classify(None, None, 256, 1.0, 0.5, 0, FAKE, None, None, None, None, None, None, None) == B.EINVAL
    clf = B.Clf(FAKE, 300)
    assert lib.disco_classify(C.byref(clf), FAKE, 256, 1.0, 0.5, 0, FAKE, None, None, None, None, None, None, None) == B.EINVAL
    assert lib.disco_classify(None, FAKE, 256, 1.0, 0.5, 0, FAKE, None, None, None, None, None, FAKE + 16, None) == B.EINVAL
    # the allocation-free form refuses a vocabulary beyond its array before any GPU call
    assert lib.disco_classify_static(None, FAKE, 65537, 1.0, 0.5, 0, FAKE, None, None, None, None, None, None) == B.ECAP
    assert b"scratch array" in lib.disco_last_error()
    assert lib.disco_draft_loop(m, kv, None, FAKE, 1, 16, 0, 1.0, 0.5, None, FAKE, FAKE, FAKE, None, FAKE, ws, None) == B.ECAP
    assert lib.disco_draft_loop(m, kv, None, FAKE, 3, 4, 0, 1.0, 0.5, None, FAKE, FAKE, FAKE, None, FAKE, ws, None) == B.EINVAL
    assert lib.disco_pack_weight(FAKE, 17, 32, FAKE, None) == B.EINVAL
    assert lib.disco_pack_weight(FAKE, 16, 40, FAKE, None) == B.EINVAL
    assert lib.disco_kv_len(kv) == 0                         # nothing advanced the cache
    lib.disco_kv_destroy(kv)
    lib.disco_model_destroy(m)
    lib.disco_model_destroy(other)


def test_sampling_and_loop_options_reject_bad_arguments_before_any_launch():
    rc, m = _model()
    lib = B.lib()
    rc, kv, _ = _kv(m)
    ws = lib.disco_workspace_bytes(m, 16, 48)
    # disco_sample: temperature, vocabulary, stride, pointers
    assert lib.disco_sample(FAKE, 1, 256, 256, 0.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 1, 256, 256, -1.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 1, 254, 256, 1.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 1, 256, 128, 1.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 0, 256, 256, 1.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(None, 1, 256, 256, 1.0, FAKE, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 1, 256, 256, 1.0, None, None, FAKE, None) == B.EINVAL
    assert lib.disco_sample(FAKE, 1, 70000, 70000, 1.0, FAKE, None, FAKE, None) == B.EINVAL
    # disco_accept_sample: block length, missing draft rows for a block with draft tokens, temperature
    assert lib.disco_accept_sample(FAKE, 0, None, FAKE, FAKE, 256, 1.0, FAKE, FAKE, FAKE, None, None) == B.ECAP
    assert lib.disco_accept_sample(FAKE, 17, None, FAKE, FAKE, 256, 1.0, FAKE, FAKE, FAKE, None, None) == B.ECAP
    assert lib.disco_accept_sample(FAKE, 3, None, None, FAKE, 256, 1.0, FAKE, FAKE, FAKE, None, None) == B.EINVAL
    assert lib.disco_accept_sample(FAKE, 3, None, FAKE, FAKE, 256, 0.0, FAKE, FAKE, FAKE, None, None) == B.EINVAL
    assert lib.disco_accept_sample(FAKE, 3, None, FAKE, FAKE, 256, 1.0, FAKE, None, FAKE, None, None) == B.EINVAL
    assert lib.disco_accept_sample(FAKE, 3, None, FAKE, FAKE + 4, 256, 1.0, FAKE, FAKE, FAKE, None, None) == B.EINVAL
    # sampled draft loop: needs uniforms, a positive temperature and a place for the probability rows
    args_tail = (FAKE, FAKE, FAKE, None, FAKE, ws, None)
    assert lib.disco_draft_loop_sampled(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, 1.0, None, FAKE, *args_tail) == B.EINVAL
    assert lib.disco_draft_loop_sampled(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, 0.0, FAKE, FAKE, *args_tail) == B.EINVAL
    assert lib.disco_draft_loop_sampled(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, 1.0, FAKE, None, *args_tail) == B.EINVAL
    # options: sampling excludes forced and reference tokens; misaligned reference pointer
    o = B.LoopOpts(None, FAKE, 1.0, FAKE, FAKE)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, FAKE + 2, 0.0, None, None)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 16, 0, 1.0, 0.5, None, *args_tail) == B.ECAP
    # the perplexity rule: threshold >= 0, and not together with a static lookahead, reference tokens or sampling
    o = B.LoopOpts(None, None, 0.0, None, None, -1.0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, None, 0.0, None, None, float("nan"))
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, None, 0.0, None, None, 20.0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 4, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, FAKE, 0.0, None, None, 20.0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, None, 1.0, FAKE, FAKE, 20.0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    assert lib.disco_kv_len(kv) == 0
    lib.disco_kv_destroy(kv)
    lib.disco_model_destroy(m)


def test_iteration_driver_and_block_continuation_reject_bad_arguments_before_any_launch():
    rc, m = _model()
    lib = B.lib()
    rc, kv, _ = _kv(m)
    rc, kv2, _ = _kv(m)
    ws = lib.disco_workspace_bytes(m, 16, 48)
    bufs = B.IterBuffers(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE)
    res = B.IterResult()
    pend = (C.c_int32 * 3)(1, 2, 3)

    def it(target=m, kv_t=kv, draft=m, kv_d=kv2, n_pending=1, cap=4, static_sl=0, chunk=0, opts=None, buffers=bufs, result=res):
        return lib.disco_iterate(target, kv_t, FAKE, ws, draft, kv_d, FAKE, ws, None, pend, n_pending, cap, static_sl, chunk,
                                 1.0, 0.5, C.byref(opts) if opts is not None else None,
                                 C.byref(buffers) if buffers is not None else None,
                                 C.byref(result) if result is not None else None, None)

    assert it(target=None) == B.EINVAL
    assert it(buffers=None) == B.EINVAL and it(result=None) == B.EINVAL
    assert it(n_pending=0) == B.EINVAL and it(n_pending=3) == B.EINVAL
    assert it(cap=-1) == B.ECAP and it(cap=16) == B.ECAP
    assert it(chunk=-1) == B.EINVAL
    assert it(buffers=B.IterBuffers(FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE)) == B.EINVAL      # no loop record
    assert it(buffers=B.IterBuffers(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None)) == B.EINVAL      # no pinned accept record
    assert it(buffers=B.IterBuffers(None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE)) == B.EINVAL      # drafting needs the token slots
    assert it(kv_d=None) == B.EINVAL
    # sampling and continuation are not options of an iteration
    assert it(opts=B.LoopOpts(None, None, 1.0, FAKE, FAKE, 0.0, 0, 0)) == B.EINVAL
    assert it(opts=B.LoopOpts(None, None, 0.0, None, None, 0.0, 2, 0)) == B.EINVAL
    assert it(opts=B.LoopOpts(None, None, 0.0, None, None, 0.0, 0, 1)) == B.EINVAL
    # continued blocks: offset + cap must fit a block, one token in, no sampling
    args_tail = (FAKE, FAKE, FAKE, None, FAKE, ws, None)
    o = B.LoopOpts(None, None, 0.0, None, None, 0.0, -1, 0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.ECAP
    o = B.LoopOpts(None, None, 0.0, None, None, 0.0, 8, 0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 8, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.ECAP
    o = B.LoopOpts(None, None, 0.0, None, None, 0.0, 2, 0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 2, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    o = B.LoopOpts(None, None, 1.0, FAKE, FAKE, 0.0, 2, 0)
    assert lib.disco_draft_loop_ex(m, kv, None, FAKE, 1, 4, 0, 1.0, 0.5, C.byref(o), *args_tail) == B.EINVAL
    assert lib.disco_kv_len(kv) == 0 and lib.disco_kv_len(kv2) == 0
    lib.disco_kv_destroy(kv)
    lib.disco_kv_destroy(kv2)
    lib.disco_model_destroy(m)


def test_kv_capacity_is_enforced_on_the_host():
    rc, m = _model(family=0)
    lib = B.lib()
    rc, kv, _ = _kv(m, capacity=16, page=16)
    ws = lib.disco_workspace_bytes(m, 16, 64)
    # a fill that would exceed the capacity is refused, as is a block that does not fit
    assert lib.disco_kv_fill(kv, FAKE, 17, None) == B.ECAP
    assert lib.disco_kv_len(kv) == 0
    lib.disco_kv_destroy(kv)
    lib.disco_model_destroy(m)


def test_prefill_rejects_bad_arguments_before_any_launch():
    lib = B.lib()
    rc, m = _model()                                  # family B
    rc, kv, _ = _kv(m, capacity=64, page=16)
    assert lib.disco_prefill_workspace_bytes(m, 0, 64) == 0
    assert lib.disco_prefill_workspace_bytes(m, B.PREFILL_MAX + 1, 64) == 0
    assert lib.disco_prefill_workspace_bytes(None, 16, 64) == 0
    need = lib.disco_prefill_workspace_bytes(m, 64, 64)
    assert need > lib.disco_workspace_bytes(m, 16, 64)
    assert lib.disco_prefill(m, kv, FAKE, 0, None, FAKE, need, None) == B.ECAP
    assert lib.disco_prefill(m, kv, FAKE, 65, None, FAKE, need, None) == B.ECAP       # 80 positions > capacity 64
    assert lib.disco_prefill(m, kv, None, 16, None, FAKE, need, None) == B.EINVAL
    assert lib.disco_prefill(m, kv, FAKE, 64, None, FAKE, need - 256, None) == B.EINVAL
    assert lib.disco_prefill(m, kv, FAKE + 2, 16, None, FAKE, need, None) == B.EINVAL
    assert lib.disco_kv_len(kv) == 0
    rc, ma = _model(family=0, max_pos=48)
    rc, kva, _ = _kv(ma, capacity=64, page=16)
    need_a = lib.disco_prefill_workspace_bytes(ma, 64, 64)
    assert lib.disco_prefill(ma, kva, FAKE, 64, None, FAKE, need_a, None) == B.ECAP    # learned position table of 48 rows
    assert "position" in B.last_error()
    assert lib.disco_prefill(m, kva, FAKE, 16, None, FAKE, need, None) == B.ESTATE     # cache of another model
    rc, mo = _model(family=0, d_ff=96)                     # family A: d_ff itself must be a multiple of 64
    rc, kvo, _ = _kv(mo, capacity=64, page=16)
    assert lib.disco_prefill(mo, kvo, FAKE, 16, None, FAKE, lib.disco_prefill_workspace_bytes(mo, 16, 64), None) == B.EINVAL
    lib.disco_kv_destroy(kvo)
    lib.disco_model_destroy(mo)
    for h in (kv, kva):
        lib.disco_kv_destroy(h)
    for h in (m, ma):
        lib.disco_model_destroy(h)


def test_prefill_workspace_grows_only_where_a_matrix_is_cut_along_k():
    """Sums of K ranges take workspace where some prompt up to the length has a matrix that is cut, and none in a model whose K
    never allows a cut; a longer prompt's workspace serves every shorter one; and what the call demands is the size without it."""
    lib = B.lib()
    rc, narrow = _model(d_model=448, n_heads=7, n_kv_heads=7, d_ff=448, vocab=256)          # 14 k-tiles
    sizes = [lib.disco_prefill_workspace_bytes(narrow, n, 64) for n in (16, 32, 48)]
    assert sizes[2] - sizes[1] == sizes[1] - sizes[0] and sizes[0] < 8 << 20
    rc, wide = _model(d_model=5120, n_heads=40, n_kv_heads=40, d_head=128, d_ff=13824, vocab=32000)
    sizes = [lib.disco_prefill_workspace_bytes(wide, n, 4096) for n in range(1, 3000, 16)]
    assert all(b >= a for a, b in zip(sizes, sizes[1:]))
    rc, kv, _ = _kv(wide, capacity=64)
    assert lib.disco_prefill(wide, kv, FAKE, 33, None, FAKE, 4096, None) == B.EINVAL
    need = int(re.search(r"(\d+) needed", B.last_error()).group(1))
    full = lib.disco_prefill_workspace_bytes(wide, 33, 48)
    assert 0 < full - need <= 64 << 20
    for h in (narrow, wide):
        for flags in (0, B.PREFILL_BF16_ACTIVATIONS):
            cut = any(c > 100 for n in range(1, 3000, 16) for c in list(B.disco_prefill_plan(h, n, flags).values())[:4])
            assert cut == (h is wide)
    lib.disco_kv_destroy(kv)
    for h in (narrow, wide):
        lib.disco_model_destroy(h)


def test_tile_cases_cover_the_launch_rule_of_the_prompt_pass():
    """Every (epilogue, tile or K ranges, precision) that the rule chooses for the model shapes of the workloads at 1 .. 3001
    tokens has a case in test_gpu_prefill.py that runs it, and the rule still chooses there what the case says."""
    from test_gpu_prefill import TILE_CASES
    code = lambda c: "s" if c > 100 else c  # noqa: E731

    def choices(shape, n, flags, handle):
        plan, gelu = B.disco_prefill_plan(handle, n, flags), "gelu" if shape.family == "A" else "swiglu"
        epi = {"qkv": "qkv", "o": "residual", "mlp_in": gelu, "mlp_out": "residual"}
        return plan, {(epi[k], code(plan[k]), bool(flags)) for k in epi}

    def handle_of(s):
        rc, h = _model(family=0 if s.family == "A" else 1, n_layers=1, d_model=s.d_model, n_heads=s.n_heads, d_head=s.d_head,
                       n_kv_heads=s.n_kv_heads, d_ff=s.d_ff, vocab=512, max_pos=8192)
        assert rc == 0
        return h

    covered, chosen = set(), set()
    for shape, pre, n, *want in TILE_CASES:
        h = handle_of(shape)
        for flags in (0, B.PREFILL_BF16_ACTIVATIONS):
            plan, triples = choices(shape, n, flags, h)
            for what, c in want[1 if flags else 0].items():
                assert code(plan[what]) == c, (shape, n, flags, plan)
            covered |= triples
        B.lib().disco_model_destroy(h)
    gqa = W.ModelShape("B", 4, 2048, 16, 128, 4, 5632, 32000)
    for shape in (W.CFG0_TARGET, W.CFG1_DRAFT, W.CFG2_TARGET, W.CFG3_TARGET, W.CFG3_DRAFT, gqa):
        h = handle_of(shape)
        for n in range(1, 3002, 16):
            for flags in (0, B.PREFILL_BF16_ACTIVATIONS):
                chosen |= choices(shape, n, flags, h)[1]
        B.lib().disco_model_destroy(h)
    assert len(chosen) >= 30 and not chosen - covered, chosen - covered


def test_tile_cases_cover_copy_rings_and_the_source_of_the_norm():
    """The finer key of the same rule: (epilogue, tile or K ranges, precision, stages of the copy ring, who forms 1 / rms, in the launch or
    one before it; none in models of LayerNorms and for matrices that read no normalised row)."""
    from test_gpu_prefill import MORE_TILE_CASES, TILE_CASES

    def keys(shape, lengths):
        rc, h = _model(family=0 if shape.family == "A" else 1, n_layers=1, d_model=shape.d_model, n_heads=shape.n_heads, d_head=shape.d_head,
                       n_kv_heads=shape.n_kv_heads, d_ff=shape.d_ff, vocab=512, max_pos=8192)
        assert rc == 0
        out, fam_b = set(), shape.family == "B"
        epi = {"qkv": "qkv", "o": "residual", "mlp_in": "swiglu" if fam_b else "gelu", "mlp_out": "residual"}
        for n in lengths:
            for flags in (0, B.PREFILL_BF16_ACTIVATIONS):
                p = B.disco_prefill_plan(h, n, flags)
                out |= {(e, "s" if p[k] > 100 else p[k], bool(flags), p["stages"][k], p["rms_in_launch"].get(k) if fam_b else None) for k, e in epi.items()}
        B.lib().disco_model_destroy(h)
        return out

    gqa = W.ModelShape("B", 4, 2048, 16, 128, 4, 5632, 32000)
    chosen = set().union(*(keys(s, range(1, 3002, 16)) for s in (W.CFG0_TARGET, W.CFG1_DRAFT, W.CFG2_TARGET, W.CFG3_TARGET, W.CFG3_DRAFT, gqa)))
    covered = set().union(*(keys(shape, [n]) for shape, pre, n, *_ in TILE_CASES + MORE_TILE_CASES))
    assert len(chosen) >= 55 and not chosen - covered, chosen - covered


@pytest.mark.parametrize("nh, nkv, dh", [(40, 40, 128), (48, 1, 128), (32, 8, 64), (32, 1, 64)])
def test_tiled_prompt_attention_only_where_a_page_offset_fits_32_bits(nh, nkv, dh):
    """The tiled kernel's offsets inside a page are 32-bit numbers of elements: a page of 2^32 elements or more (a cache kept as
    one page is accepted, whatever its size) has to go to the general kernel, whose offsets are 64 bits wide."""
    rc, m = _model(n_heads=nh, n_kv_heads=nkv, d_head=dh)
    assert rc == 0
    tiled = []
    for log2 in range(3, 28):
        pt = 1 << log2
        if B.disco_prefill_plan(m, 2048, page_tokens=pt)["attn_tiles"]:
            tiled.append(pt)
            # the last element a lane may address: the last token of the last channel of the last head's V block
            assert (2 * nkv - 1) * pt * dh + (dh - 1) * pt + pt - 1 < 1 << 32, pt
    assert tiled[0] == 8 and len(tiled) >= 10
    B.lib().disco_model_destroy(m)


@pytest.mark.parametrize("family, nh, nkv, dh, per_head", [
    (1, 12, 12, 64, 6), (1, 4, 4, 64, 6), (1, 40, 40, 128, 6), (1, 20, 20, 128, 12), (1, 80, 80, 64, 3), (1, 48, 48, 128, 0),
    (1, 35, 35, 128, 6), (1, 50, 25, 128, 0), (1, 16, 4, 128, 0), (1, 6, 2, 64, 0), (0, 12, 1, 64, 0), (0, 48, 1, 128, 0), (0, 12, 12, 64, 0)])
def test_the_deal_of_the_context_does_not_depend_on_the_launch(family, nh, nkv, dh, per_head):
    """The deal decides the order in which the attention adds up, so it is a function of the model and the length alone: a
    `per_head`-th of the context, 128 positions at least and in steps of 32, in models with K / V heads of their own whose
    projection has at most 256 workgroups (per_head of them for each head); one, 128, 256, 512 or 1024 positions a range elsewhere."""
    rc, m = _model(family=family, n_heads=nh, n_kv_heads=nkv, d_head=dh)
    assert rc == 0
    gemm = (nh + 2 * nkv) * dh
    rows = 64 if gemm % 64 == 0 and gemm // 64 >= 200 else 32
    for ctx in list(range(0, 1700, 7)) + [255, 256, 2475, 4000, 6000]:
        for n in (1, 6, 16):
            total = ctx + n
            if per_head:
                want = max(128, -(-(-(-total // per_head)) // 32) * 32)
            else:
                want = next(l for most, l in ((256, 256), (768, 128), (1536, 256), (3072, 512), (1 << 30, 1024)) if total <= most)
            ranges = -(-total // want)
            plan = B.disco_qkv_attn_plan(m, n, ctx, 256)
            assert (plan["range"], plan["ranges"], plan["row_tiles"]) == (want, ranges, rows // 16), (total, plan)
            own = gemm // rows + nh * (1 if total <= 256 else ranges)
            form = "own" if rows == 32 and own <= 256 else ("shared" if per_head and total > 256 else "separate")
            assert plan["form"] == form and plan["workgroups"] == {"own": own, "shared": gemm // rows, "separate": 0}[form], (total, plan)
    B.lib().disco_model_destroy(m)


def test_heuristic_lookahead_rule_by_hand():
    """The acceptance-following lookahead rule (the reading of the paper's unnamed heuristic: +up after a fully
    accepted block, -down otherwise, inside [1, cap]; nothing drafted: unchanged), on hand cases and on the
    hand sequence that pins the oracle's heuristic policy."""
    f = B.disco_heuristic_next
    assert f(5, 5, 5, 2, 1, 10) == 7 and f(9, 9, 9, 2, 1, 10) == 10 and f(10, 10, 10, 2, 1, 10) == 10
    assert f(5, 5, 4, 2, 1, 10) == 4 and f(1, 1, 0, 2, 1, 10) == 1 and f(2, 2, 0, 2, 3, 10) == 1
    assert f(5, 0, 0, 2, 1, 10) == 5 and f(12, 0, 0, 2, 1, 10) == 10
    # start 5: full, full, full (cap 10), reject, reject, full
    sl, seen = 5, []
    for drafted_all in (True, True, True, False, False, True):
        seen.append(sl)
        sl = f(sl, sl, sl if drafted_all else 0, 2, 1, 10)
    assert seen == [5, 7, 9, 10, 9, 8] and sl == 10
    for bad in ((0, 1, 1, 2, 1, 10), (5, 2, 3, 2, 1, 10), (5, 2, 1, -1, 1, 10), (5, 2, 1, 2, 1, 0)):
        with pytest.raises(B.DiscoError) as e:
            f(*bad)
        assert e.value.code == B.EINVAL
    lib = B.lib()
    assert lib.disco_clf_examples(None, 4, FAKE, FAKE, FAKE, None, None) == B.EINVAL
    assert lib.disco_clf_examples(FAKE, 0, FAKE, FAKE, FAKE, None, None) == B.EINVAL


def test_bench_reads_the_measured_traffic_of_both_configurations_from_profiles():
    """bench.py takes `roofline.traffic` from the counter summaries under profiles/ (never from a literal): the
    summaries must be there, carry the line it parses, and sit within a few per cent above the algorithmic bytes."""
    import importlib.util
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    gate_up = 2 * 13824 * 5120 * 2              # 13B-class gate + up, bf16
    w1 = 24576 * 6144 * 2                       # 15B-class W1, bf16
    for cfg, panels, algorithmic in (("cfg4", 1, gate_up), ("cfg4", 2, gate_up), ("cfg3", 1, w1)):
        t = bench.gateup_traffic_bytes(panels, cfg)
        assert t is not None and algorithmic <= t <= 1.05 * algorithmic, (cfg, panels, t)
