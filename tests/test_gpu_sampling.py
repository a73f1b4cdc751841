"""GPU parity of the sampling path (temperature > 0): draws by inverse CDF, speculative-sampling
acceptance, and the loop built on them, against the CPU oracle on the same logits and the same
uniforms.

Floating point decides integers here (which CDF interval holds u * total; whether u q < p), so the
comparison is exact except where the oracle reports that the decision is within rounding of its
boundary: a draw whose target lies closer than DRAW_MARGIN (as a fraction of the total) to an interval
boundary, a keep / reject test with |u q - p| / q below ACC_MARGIN.  The GPU sums in fp32 (segment
by segment, 64-lane scans), the oracle in float64 in index order; both follow the same definition."""
import numpy as np
import pytest
import torch

from paper_2405_04304_amd import binding as B
from paper_2405_04304_amd.engine import SpecEngine
from oracle import disco_oracle as O
from workloads import synth as W

pytestmark = pytest.mark.gpu

DRAW_MARGIN = 2e-5
ACC_MARGIN = 1e-4


def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def _gpu_sample(logits, T, u, ld=None, want_probs=True):
    d = dev()
    rows, V = logits.shape
    ld = ld or V
    buf = torch.zeros(rows, ld, dtype=torch.float32, device=d)
    buf[:, :V] = logits.to(d)
    probs = torch.full((rows, V), -1.0, dtype=torch.float32, device=d) if want_probs else None
    toks = torch.full((rows,), -7, dtype=torch.int32, device=d)
    B.disco_sample(buf, rows, V, ld, T, u.to(d), probs, toks)
    torch.cuda.synchronize()
    return toks.cpu().tolist(), (probs.cpu() if want_probs else None)


@pytest.mark.parametrize("V", [16, 1000, 4096, 32000, 49152, 65536])
def test_sample_rows_match_oracle(V):
    g = torch.Generator().manual_seed(V)
    rows = 6
    for T, sigma in ((1.0, 2.0), (0.7, 0.5), (2.0, 4.0)):
        logits = (torch.randn(rows, V, generator=g) * sigma).to(torch.float32)
        u = W.make_uniforms(V + int(T * 10), rows, "sample")
        toks, probs = _gpu_sample(logits, T, u, ld=V + 8 if V % 8 == 0 else None)
        n_flag = 0
        for r in range(rows):
            p = O.softmax_t(logits[r], T)
            assert torch.allclose(probs[r].double(), p, rtol=2e-4, atol=1e-12), (V, T, r)
            assert abs(float(probs[r].double().sum()) - 1.0) < 1e-4
            want, margin = O.sample_index(p, float(u[r]))
            if toks[r] != want:
                assert margin < DRAW_MARGIN, (V, T, r, toks[r], want, margin)
                assert abs(toks[r] - want) <= 2
                n_flag += 1
        assert n_flag <= 1
    # end points and degenerate rows
    logits = torch.zeros(4, V, dtype=torch.float32)
    logits[1, V // 3] = 80.0                    # one-hot after the softmax
    logits[2, :] = -1e4; logits[2, 5] = 0.0; logits[2, V - 3] = 0.0      # two tokens share the mass
    logits[3, :] = 3.0                          # uniform: token floor(u V)
    u = torch.tensor([0.0, 0.77, 0.75, 0.4321], dtype=torch.float32)
    toks, probs = _gpu_sample(logits, 1.0, u)
    assert toks[0] == 0 and toks[1] == V // 3 and toks[2] == V - 3
    want3, margin3 = O.sample_index(torch.ones(V, dtype=torch.float64), float(u[3]))
    assert toks[3] == want3 or margin3 < DRAW_MARGIN
    assert float(probs[2][5]) == pytest.approx(0.5) and float(probs[2][7]) == 0.0


@pytest.mark.parametrize("V", [4096, 32000, 49152, 65536])
def test_probability_rows_keep_the_precision_of_expf(V):
    """Logits on a grid of 2^-10 below a maximum of 0: x - max and the division by T = 1 are exact and the largest probability is
    1 / S itself, so p_i / p_max differs from e^x_i by the exponential's rounding and one product's.  A correct rounding of a
    value with a log-uniform mantissa has a relative rms error of 2^-23 / sqrt(12) * sqrt(0.541) = 2.53e-8, two of them 3.58e-8;
    the bar is 12 % above (expf measures 3.6e-8, a shorter form of 1.5 ulp 4.4e-8)."""
    g = torch.Generator().manual_seed(V)
    logits = -torch.randint(0, 16 * 1024, (3, V), generator=g).to(torch.float32) / 1024
    logits[:, 7] = 0.0
    _, probs = _gpu_sample(logits, 1.0, torch.full((3,), 0.5))
    got, want = probs.double() / probs[:, 7:8].double(), logits.double().exp()
    rms = float((((got - want) / want) ** 2).mean().sqrt())
    print(f"[sampling] V {V}: rms error of p / p_max {rms:.2e}", flush=True)
    assert rms <= 4e-8


@pytest.mark.parametrize("V", [4096, 32000, 49152, 65536])
def test_row_sums_are_pairwise(V):
    """The largest probability of such rows is 1 / S: the rounding of S and of its reciprocal.  A sum whose parts are of like size at
    every level of a tree gathers sqrt(1 + 1/2 + 1/4 + ..) = sqrt(2) roundings of 2.53e-8 rms, with the reciprocal's sqrt(3): 4.4e-8;
    the bar is 25 % above.  (Lane and wavefront sums one after another: 6.0e-8 .. 6.9e-8.)"""
    g = torch.Generator().manual_seed(V + 1)
    logits = -torch.randint(0, 16 * 1024, (300, V), generator=g).to(torch.float32) / 1024
    logits[:, 7] = 0.0
    _, probs = _gpu_sample(logits, 1.0, torch.full((300,), 0.5))
    err = probs[:, 7].double() * logits.double().exp().sum(1) - 1.0
    print(f"[sampling] V {V}: rms error of 1 / S {float(err.square().mean().sqrt()):.2e}", flush=True)
    assert float(err.square().mean().sqrt()) <= 5.5e-8


def test_subnormal_weights_are_weights():
    """e^-95 and e^-100 are subnormal in fp32 and not zero: the row stores them, a draw at 0 takes the first of them, and a
    drafted token of such a probability is kept at u = 0."""
    V = 4096
    logits = torch.full((1, V), -300.0)
    logits[0, 3], logits[0, 1234], logits[0, 4000] = -100.0, -95.0, 0.0
    toks, probs = _gpu_sample(logits, 1.0, torch.zeros(1))
    assert toks == [3]
    want = logits.double().exp()
    for i in (3, 1234):                                   # half a step of the subnormals (2^-149) for each of two roundings
        assert abs(float(probs[0, i].double() - want[0, i])) <= 2.0 ** -149
    q = [torch.nn.functional.one_hot(torch.tensor(1234), V).to(torch.float32)]
    n, emit = _gpu_accept(torch.cat([logits, logits]), q, [0, 1234], torch.zeros(1), torch.tensor([0.5, 0.5]), 1.0)
    assert (n, emit) == (1, [1234, 4000])


def _accept_case(g, V, sl, T, mode):
    """Random block: target logits, draft rows near the target (so that keeps and rejections both occur)."""
    lt = torch.from_numpy(g.normal(size=(sl + 1, V)) * 2.0).to(torch.float32)
    if mode == "same":
        ld = lt[:sl].clone()
    elif mode == "far":
        ld = torch.from_numpy(g.normal(size=(sl, V)) * 2.0).to(torch.float32)
    else:
        ld = lt[:sl] + torch.from_numpy(g.normal(size=(sl, V)) * 0.5).to(torch.float32)
    q_rows = [O.softmax_t(ld[j], T).to(torch.float32) for j in range(sl)]       # fp32 rows, shared by both sides
    block = [int(g.integers(0, V))] + [O.sample_index(q_rows[j], float(g.random()))[0] for j in range(sl)]
    u_acc = torch.from_numpy(g.random(max(sl, 1)).astype(np.float32))
    u_res = torch.from_numpy(g.random(sl + 1).astype(np.float32))
    return lt, q_rows, block, u_acc, u_res


def _gpu_accept(lt, q_rows, block, u_acc, u_res, T, dev_n_block=None):
    d = dev()
    V = lt.shape[1]
    q = torch.stack(q_rows).to(d) if q_rows else torch.zeros(1, V, dtype=torch.float32, device=d)
    out = B.struct_tensor(B.AcceptOut, 1, d)
    host = B.struct_tensor(B.AcceptOut, 1, pinned=True)
    blk = torch.tensor(block + [0] * (16 - len(block)), dtype=torch.int32, device=d)
    nb = None if dev_n_block is None else torch.tensor([dev_n_block], dtype=torch.int32, device=d)
    B.disco_accept_sample(blk, len(block), q, lt.to(d).contiguous(), V, T, u_acc.to(d), u_res.to(d), out, host,
                          dev_n_block=nb)
    torch.cuda.synchronize()
    a, h = B.read_struct(B.AcceptOut, out), B.AcceptOut.from_buffer_copy(host.numpy().tobytes())
    assert (a.n, a.n_emit, list(a.emit)) == (h.n, h.n_emit, list(h.emit))
    return a.n, list(a.emit[:a.n_emit])


@pytest.mark.parametrize("V", [252, 32000, 65536])
def test_accept_sample_with_the_block_inside_the_record(V):
    """The record may be written over the block it was made from: the same outcome as with buffers apart, for blocks that are kept
    whole, rejected at once and in between, at every offset of the block in the record that lies on a word."""
    d = dev()
    for sl, mode, shift in ((0, "near", 0), (3, "same", 2), (6, "near", 1), (9, "far", 2), (12, "near", 3), (15, "same", 2)):
        lt, q_rows, block, u_acc, u_res = _accept_case(np.random.default_rng(V + sl), V, sl, 1.0, mode)
        want = _gpu_accept(lt, q_rows, block, u_acc, u_res, 1.0)
        buf = torch.zeros(18 + 16, dtype=torch.int32, device=d)         # the record's 18 words and room for a block that sticks out
        buf[shift:shift + sl + 1] = torch.tensor(block, dtype=torch.int32, device=d)
        q = torch.stack(q_rows).to(d) if q_rows else torch.zeros(1, V, dtype=torch.float32, device=d)
        B.disco_accept_sample(buf[shift:], sl + 1, q, lt.to(d).contiguous(), V, 1.0, u_acc.to(d), u_res.to(d), buf)
        torch.cuda.synchronize()
        got = buf[:18].cpu().tolist()
        assert (got[0], got[2:2 + got[1]]) == want and got[1] == got[0] + 1 and got[2 + got[1]:] == [-1] * (16 - got[1]), (sl, mode, shift)


@pytest.mark.parametrize("V", [4, 252, 256, 260, 4092, 4100, 8192, 8196, 32768, 32772, 49152, 49156, 65536])
def test_row_kernels_at_segment_edges(V):
    """A row is dealt to sixteen wavefronts in segments of 256, in templates of 2 / 8 / 12 / 16 segments: lengths around the
    edges, and draws that fall on the first and last elements (point masses: the answer needs no tolerance)."""
    ids = sorted({0, 3, V // 2, V - 4, V - 1} | {i for i in (255, 256, 4095, 4096) if i < V})
    logits = torch.full((len(ids), V), -200.0)
    for r, i in enumerate(ids):
        logits[r, i] = 0.0
    for u in (0.0, 0.5, 1.0 - 2.0 ** -24):
        toks, probs = _gpu_sample(logits, 1.0, torch.full((len(ids),), u))
        assert toks == ids and torch.equal(probs, (logits == 0).to(torch.float32))
    # one block per outcome: rows whose draft token is the target's are kept, the first other row draws the target's token
    rows = min(len(ids), 6)
    q = [torch.nn.functional.one_hot(torch.tensor(i), V).to(torch.float32) for i in ids[:rows - 1]]
    lt = logits[:rows]
    u_acc, u_res = torch.full((rows - 1,), 0.5), torch.full((rows,), 0.25)
    n, emit = _gpu_accept(lt, q, [1] + ids[:rows - 1], u_acc, u_res, 1.0)
    assert n == rows - 1 and emit == ids[:rows]
    if rows > 2:
        k = rows // 2
        q[k - 1] = torch.nn.functional.one_hot(torch.tensor(ids[k]), V).to(torch.float32)
        block = [1] + ids[:k - 1] + [ids[k]] + ids[k:rows - 1]
        n, emit = _gpu_accept(lt, q, block, u_acc, u_res, 1.0)
        assert n == k - 1 and emit == ids[:k]
        n, emit = _gpu_accept(lt, q, block, u_acc, u_res, 1.0, dev_n_block=k)      # only the rows before the rejected one
        assert n == k - 1 and emit == ids[:k]


def test_accept_sample_matches_oracle():
    g = np.random.default_rng(5)
    n_cmp = n_flag = 0
    seen_n = set()
    for V in (512, 4096, 32000):
        for sl in (0, 1, 2, 5, 10, 15):
            for mode in ("near", "same", "far"):
                for T in ((1.0,) if V == 32000 else (1.0, 0.6)):
                    lt, q_rows, block, u_acc, u_res = _accept_case(g, V, sl, T, mode)
                    p_rows = [O.softmax_t(lt[j], T) for j in range(sl + 1)]
                    n, emit, info = O.accept_stochastic(block, q_rows, p_rows, u_acc.tolist(), u_res.tolist())
                    gn, gemit = _gpu_accept(lt, q_rows, block, u_acc, u_res, T)
                    flagged = any(m < ACC_MARGIN for m in info["accept_margins"]) or info["sample_margin"] < DRAW_MARGIN
                    n_cmp += 1
                    if (gn, gemit) != (n, emit):
                        assert flagged, (V, sl, mode, T, gn, n, gemit, emit, info)
                        n_flag += 1
                    if mode == "same" and not flagged:
                        assert gn == sl                     # identical distributions: nothing is rejected
                    seen_n.add((sl, n))
    assert n_flag <= 2, n_flag
    assert any(n < sl for sl, n in seen_n) and any(n == sl and sl > 0 for sl, n in seen_n)
    print(f"[parity] accept_sample: {n_cmp} blocks, {n_flag} at a flagged decision", flush=True)
    # a draft token the target excludes is rejected at once and cannot be re-drawn
    V = 512
    lt = torch.full((2, V), -1e4, dtype=torch.float32); lt[:, 7] = 0.0; lt[:, 9] = 1.0
    q = torch.zeros(V, dtype=torch.float32); q[3] = 0.5; q[9] = 0.5
    # p = (0.269 at token 7, 0.731 at token 9); residual max(0, p - q) = (0.269, 0.231), total 0.5
    for u_r, want in ((0.25, 7), (0.9, 9)):
        gn, gemit = _gpu_accept(lt, [q], [1, 3], torch.tensor([0.5]), torch.tensor([u_r, 0.5]), 1.0)
        on, oemit, _ = O.accept_stochastic([1, 3], [q], [O.softmax_t(lt[j], 1.0) for j in range(2)], [0.5], [u_r, 0.5])
        assert (gn, gemit) == (0, [want]) == (on, oemit)
    # a device-resident block length shortens the block
    g2 = np.random.default_rng(9)
    lt, q_rows, block, u_acc, u_res = _accept_case(g2, 4096, 6, 1.0, "same")
    gn, gemit = _gpu_accept(lt, q_rows, block, u_acc, u_res, 1.0, dev_n_block=3)
    on, oemit, _ = O.accept_stochastic(block[:3], q_rows[:2], [O.softmax_t(lt[j], 1.0) for j in range(3)], u_acc.tolist(), u_res.tolist())
    assert (gn, gemit) == (on, oemit) and gn == 2


def _flagged(it, tau):
    if it["sample_margin"] < DRAW_MARGIN or any(m < ACC_MARGIN for m in it["accept_margins"]):
        return True
    for st in it["steps"]:
        if st["sample_margin"] < DRAW_MARGIN:
            return True
        if tau is not None and abs(st["score"] - tau) < 1e-3:
            return True
    return False


def _compare_sampling_runs(gpu, orc, tau):
    """Iterations must agree one by one; a difference is allowed only in an iteration the oracle flags,
    and ends the comparison (the two texts are different random walks from there on)."""
    for k, (gi, oi) in enumerate(zip(gpu["iterations"], orc["iterations"])):
        same = (gi["sl"], gi["n"], gi["block"], gi["emit"]) == (oi["sl"], oi["n"], oi["block"], oi["emit"])
        if not same:
            assert _flagged(oi, tau), (k, gi, {x: oi[x] for x in ("sl", "n", "block", "emit")})
            return k
    assert gpu["tokens"] == orc["tokens"]
    return None


def test_sampling_loop_matches_oracle():
    d = dev()
    n_new = 48
    cases = []
    # tiny pre-LN pair (early-exit draft) and a small rotary pair with an independent draft
    tw = W.make_weights(W.CFG0_TARGET, 0, "bf16")
    cases.append((W.CFG0_TARGET, W.CFG0_DRAFT, tw, W.early_exit_draft(tw, 1), 32))
    st = W.ModelShape("B", 2, 128, 2, 64, 2, 256, 512)
    sd = W.ModelShape("B", 1, 128, 2, 64, 2, 256, 512)
    w_t = W.make_weights(st, 0, "bf16", sigma=0.1)
    w_d = {k: v.clone() for k, v in W.make_weights(sd, 10, "bf16", sigma=0.1).items()}
    for k in ("tok_emb", "wlm", "normf_g"):          # a related draft: the target's tables, its own layer
        w_d[k] = w_t[k]
    cases.append((st, sd, w_t, w_d, 40))
    clf = W.make_classifier(100)
    n_div = n_runs = 0
    for shape_t, shape_d, wt, wd, n_prompt in cases:
        ot, od = O.Model(shape_t, wt, kv_bf16=True), O.Model(shape_d, wd, kv_bf16=True)
        prompt = W.make_prompt(1, n_prompt, shape_t.vocab).tolist()
        eng = SpecEngine(B.DiscoModel(shape_t, wt, d), B.DiscoModel(shape_d, wd, d), B.DiscoClf(clf, d),
                         max_ctx=n_prompt + n_new + 16, page_tokens=8)
        for T in (1.0, 0.5):
            u = {k: W.make_uniforms(21, n_new + 16, k) for k in ("draft", "accept", "resample")}
            # (the seeded classifier's score grows with the position feature: at tau 0.6 early iterations
            # halt after one token and later ones run to the cap)
            for pol in ({"mode": "static", "gamma": 4}, {"mode": "disco", "tau": 0.6, "sl_max": 6, "pos_mode": "absolute"}):
                orc = O.spec_decode_sampling(ot, od, clf, prompt, n_new, pol, T, u)
                gpu = eng.generate_sampling(prompt, n_new, pol, T, u)
                assert len(gpu["tokens"]) == n_new
                n_runs += 1
                if _compare_sampling_runs(gpu, orc, pol.get("tau")) is not None:
                    n_div += 1
                acc = sum(it["n"] for it in orc["iterations"])
                assert 0 < acc < sum(it["sl"] for it in orc["iterations"])     # both outcomes occur
        # a vanishing temperature gives the GPU's own greedy text (margins permitting)
        ref, margins = O.greedy_target(ot, prompt, n_new)
        gg = eng.greedy(prompt, n_new)
        cold = eng.generate_sampling(prompt, n_new, {"mode": "static", "gamma": 3}, 1e-4, u)
        if min(margins) > 5e-3:
            assert cold["tokens"] == gg == ref
    assert n_div <= 2, (n_div, n_runs)
    print(f"[parity] sampling loop: {n_runs} runs, {n_div} left the oracle's path at a flagged decision", flush=True)
