"""Forwards on several streams at once in the default launch mode.  Launches whose workgroups wait for each other run one forward at a time on a GPU; a
forward that meets another one's takes a launch per phase, with the same bits."""
import pytest
import torch

from paper_2405_04304_amd import binding as B
from workloads import synth as W

from test_gpu_parity import dev

pytestmark = pytest.mark.gpu

# (shape, cached positions, tokens): what the forward is alone
KINDS = {
    "all layers": (W.ModelShape("A", 3, 768, 12, 64, 1, 3072, 4096), 700, 1, "layers"),
    "all layers, heads of their own": (W.ModelShape("B", 2, 768, 12, 64, 12, 3072, 4096), 523, 2, "layers"),
    "workgroups of its own": (W.ModelShape("B", 2, 256, 6, 64, 2, 512, 4096), 640, 7, "shared"),
    "whole heads": (W.ModelShape("B", 2, 256, 4, 64, 4, 512, 4096), 200, 5, "shared"),
    "shared workgroups": (W.ModelShape("B", 1, 64, 68, 64, 68, 64, 4096), 300, 3, "shared"),
}


class _Program:
    """A cache, a workspace and a stream of its own; step() sends one verification and takes its entries back."""
    def __init__(self, kind, stream, gm):
        self.shape, self.ctx, self.m, self.route = KINDS[kind]
        self.gm, self.stream = gm, stream
        self.kv, self.ws = B.DiscoKV(gm, self.ctx + 32, 16), gm.workspace(16, self.ctx + 32)
        self.kv.fill(W.make_kv_fill(self.shape, self.ctx, 3).to(dev()))
        self.blk = W.make_tokens(80, self.m, self.shape.vocab).to(torch.int32).to(dev())
        self.am = torch.zeros(16, dtype=torch.int32, device=dev())

    def step(self):
        lg = torch.full((self.m, self.shape.vocab), -7.0, device=dev())
        torch.cuda.current_stream().synchronize()                # (allocated and filled before another stream writes it)
        return self.send(lg)

    def send(self, lg):
        B.disco_verify(self.gm, self.kv, self.blk, self.m, self.am, lg, self.ws, stream=self.stream.cuda_stream)
        route = B.disco_forward_route()
        B.disco_kv_rollback(self.kv, self.ctx)
        return lg, route


def _models(kinds):
    return {k: B.DiscoModel(KINDS[k][0], W.make_weights(KINDS[k][0], 90, "bf16", sigma=0.05), dev()) for k in kinds}


@pytest.mark.parametrize("kind", list(KINDS))
def test_a_second_stream_takes_launches_that_wait_nowhere(kind):
    gm = _models([kind])[kind]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    p1, p2, p3 = _Program(kind, s1, gm), _Program(kind, s2, gm), _Program(kind, s1, gm)
    want, route = p1.step()
    assert route == KINDS[kind][3]
    out = [torch.empty_like(want) for _ in range(3)]
    torch.cuda.synchronize()
    for _ in range(2):
        with torch.cuda.stream(s1):
            torch.cuda._sleep(50_000_000)                        # holds the first stream's forwards back
        assert p1.send(out[0])[1] == route
        assert p2.send(out[1])[1] == "phases"                    # the first one is still to come
        assert p3.send(out[2])[1] == route                       # on one stream they run one after the other
        assert not s1.query()
        torch.cuda.synchronize()
        for o in out:
            assert torch.equal(o, want)
        assert p2.send(out[1])[1] == route                       # the place is free again
        torch.cuda.synchronize()
        assert torch.equal(out[1], want)
    # a gated forward gives it back too
    gate, lg = torch.ones(1, dtype=torch.int32, device=dev()), torch.empty(p1.shape.vocab, device=dev())
    B.disco_draft_step(gm, p1.kv, p1.blk, 1, lg, p1.ws, gate=gate, stream=s1.cuda_stream)
    B.disco_kv_rollback(p1.kv, p1.ctx)
    torch.cuda.synchronize()
    assert p2.send(out[1])[1] == route
    torch.cuda.synchronize()


def test_programs_on_many_streams_agree_with_one_after_the_other():
    """Eight programs of all kinds, on eight streams, thirty forwards each without a synchronisation between them."""
    kinds = list(KINDS) + ["all layers", "all layers", "all layers, heads of their own"]
    models = _models(KINDS)
    progs = [_Program(k, torch.cuda.Stream(), models[k]) for k in kinds]
    want = [p.step()[0] for p in progs]
    torch.cuda.synchronize()
    outs = [[torch.empty_like(w) for _ in range(30)] for w in want]
    torch.cuda.synchronize()
    routes = set()
    for i in range(30):
        for p, o in zip(progs, outs):
            routes.add(p.send(o[i])[1])
    torch.cuda.synchronize()
    for k, w, o in zip(kinds, want, outs):
        for i, lg in enumerate(o):
            assert torch.equal(lg, w), (k, i)
    assert "phases" in routes and len(routes) > 1


def test_a_captured_forward_holds_no_launch_of_all_layers():
    kind = "all layers"
    gm = _models([kind])[kind]
    p = _Program(kind, torch.cuda.current_stream(), gm)
    want = p.step()[0]
    lg = torch.empty_like(want)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        B.disco_verify(gm, p.kv, p.blk, p.m, p.am, lg, p.ws)
    assert B.disco_forward_route() == "shared"
    for _ in range(3):
        lg.fill_(0.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(lg, want)
        B.disco_kv_rollback(p.kv, p.ctx)
        assert torch.equal(p.step()[0], want)
        torch.cuda.synchronize()
