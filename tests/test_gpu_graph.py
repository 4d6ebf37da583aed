"""The whole step (route, paged GEMMs, combine) captured in a HIP graph and
replayed: every replay is bit-identical to the eager step, for each GEMM path
(decode kernels, streaming kernel, LDS-tiled kernel), with eager work on the
same stream between replays. Nothing in the step allocates or clears memory
with a memset, so the captured launches are the eager ones.

Layers that are large enough fork work to a stream of their own (the second
chain of the routed experts under capture, the shared experts): the last
three tests take such layers; two of them hold pages of every format and look
for the two branches in the captured graph."""
import ctypes
import dataclasses

import numpy as np
import pytest

from helpers import case, gpu_layer, gpu_random_layer, say, to_dev, to_dev16
from paper_2607_16184_amd import pw, synth
from test_gemm_plan import DECODE, STREAM, TILED, Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,chains", [(16, 2), (16, 1), (300, 2), (1000, 2)])
def test_graph_replay_matches_eager(T, chains):
    """A small layer: one stream and one graph branch, whatever the chains."""
    import torch
    from paper_2607_16184_amd.layer import PagedLayer
    cfg, w16, bits, order = case("tiny", T=T)
    say("graph replay tiny T=%d chains=%d" % (T, chains))
    L = gpu_layer(cfg, w16, bits, order)
    L.set_chains(chains)
    logits, x = to_dev(synth.logits(cfg)), to_dev16(synth.activations(cfg))
    rbuf = PagedLayer.routing_buffers(cfg.T, cfg.E, cfg.K)
    y = torch.empty((cfg.T, cfg.H), dtype=torch.float32, device="cuda")

    def step():
        L.forward(x, L.route(logits, cfg.K, out=rbuf), out_fp32=True, y=y)

    step()
    torch.cuda.synchronize()
    want = y.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    other = torch.empty_like(y)
    for r in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), r
        L.forward(x, L.route(logits, cfg.K), out_fp32=True, y=other)   # eager work in between
        torch.cuda.synchronize()
        assert torch.equal(other, want), r
    L.close()


@pytest.mark.parametrize("T", [16, 100])
def test_graph_replay_shared_experts(T):
    """A small layer with shared experts, whose GEMMs follow the routed ones on
    the caller's stream. Every replay is bit-identical to the eager step, with
    eager steps between the replays."""
    import torch
    from paper_2607_16184_amd.layer import PagedLayer
    cfg, w16, bits, order = case("tiny_shared", T=T)
    say("graph replay, shared experts, T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    L.set_shared_experts(cfg.n_shared)
    logits, x = to_dev(synth.logits(cfg)), to_dev16(synth.activations(cfg))
    gate = to_dev(synth.shared_gate(cfg))
    Kt = cfg.K + cfg.n_shared
    rbuf = PagedLayer.routing_buffers(cfg.T, cfg.E, Kt)
    y = torch.empty((cfg.T, cfg.H), dtype=torch.float32, device="cuda")

    def step(out):
        L.forward(x, L.route_shared(logits, cfg.K, cfg.n_shared, gate=gate, out=rbuf), out_fp32=True, y=out)

    step(y)
    torch.cuda.synchronize()
    want = y.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(y)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step(y)
    other = torch.empty_like(y)
    for r in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), r
        step(other)                                        # eager work in between
        torch.cuda.synchronize()
        assert torch.equal(other, want), r
    L.close()


@pytest.mark.parametrize("T", [16, 40, 100])
def test_chains_bit_identical(T):
    """The chains setting changes no bits, 16-bit and fp32 out (here, in a small
    layer, both settings launch alike), and takes 1 or 2 only."""
    import torch
    cfg, w16, bits, order = case("tiny", T=T)
    say("one chain vs two chains, tiny T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    logits, x = to_dev(synth.logits(cfg)), to_dev16(synth.activations(cfg))
    routing = L.route(logits, cfg.K)
    out = {}
    for chains in (1, 2):
        L.set_chains(chains)
        out[chains] = (L.forward(x, routing).clone(), L.forward(x, routing, out_fp32=True).clone())
    torch.cuda.synchronize()
    assert torch.equal(out[1][0], out[2][0]) and torch.equal(out[1][1], out[2][1])
    from paper_2607_16184_amd import pw
    for bad in (0, 3):
        with pytest.raises(pw.PWError) as ei:
            L.set_chains(bad)
        assert ei.value.status == pw.PW_EINVAL
    L.close()


@pytest.mark.parametrize("T,kw", [(16, {}), (100, {}), (600, dict(F=4096, n_shared=4, E=12))])
def test_chains_bit_identical_shared(T, kw):
    """The chains setting changes no bits with shared experts either (small
    layers: both settings launch alike, but for the 600-token batch of four
    shared experts, which forks call by call)."""
    import torch
    cfg, w16, bits, order = case("tiny_shared", T=T, **kw)
    say("one chain vs two chains with shared experts, T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    L.set_shared_experts(cfg.n_shared)
    logits, x = to_dev(synth.logits(cfg, T=T)), to_dev16(synth.activations(cfg, T=T))
    gate = to_dev(synth.shared_gate(cfg, T=T))
    routing = L.route_shared(logits, cfg.K, cfg.n_shared, gate=gate)
    out = {}
    for chains in (1, 2):
        L.set_chains(chains)
        out[chains] = (L.forward(x, routing).clone(), L.forward(x, routing, out_fp32=True).clone())
    torch.cuda.synchronize()
    assert torch.equal(out[1][0], out[2][0]) and torch.equal(out[1][1], out[2][1])
    L.close()


@pytest.mark.parametrize("n_shared", [0, 2])
def test_forked_layer_stream_bit_identical(n_shared):
    """A layer large enough (256 MiB of pages) for its calls to fork: the
    second expert chain under capture, the shared experts in every call. The
    graph's replays and the eager calls give the bits of one chain."""
    import torch
    from paper_2607_16184_amd.layer import PagedLayer
    E, T = 8 + n_shared, 40
    cfg, w16, _, order = case("tiny_shared", E=E, H=2048, F=2816, T=T, n_shared=n_shared)
    bits = [np.full((E, cfg.nrb(p)), 16, np.int32) for p in range(3)]
    say("forked layer stream, n_shared=%d" % n_shared)
    L = gpu_layer(cfg, w16, bits, order)
    assert L.stats()[0] >= 256 << 20
    L.set_shared_experts(n_shared)
    logits, x = to_dev(synth.logits(cfg)), to_dev16(synth.activations(cfg))
    gate = to_dev(synth.shared_gate(cfg)) if n_shared else None
    rbuf = PagedLayer.routing_buffers(T, E, cfg.K + n_shared)
    y = torch.empty((T, cfg.H), dtype=torch.float32, device="cuda")

    def step(out):
        L.forward(x, L.route_shared(logits, cfg.K, n_shared, gate=gate, out=rbuf), out_fp32=True, y=out)

    L.set_chains(1)
    step(y)
    torch.cuda.synchronize()
    want = y.clone()
    L.set_chains(2)
    step(y)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        step(y)
    other = torch.empty_like(y)
    for r in range(3):
        y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want), r
        step(other)                                        # eager work in between
        torch.cuda.synchronize()
        assert torch.equal(other, want), r
    L.close()


def _branches(graph):
    """Whether some node of a captured graph has two successors."""
    n = ctypes.c_size_t(0)
    raw = ctypes.c_void_p(graph.raw_cuda_graph())
    assert pw._lib.hipGraphGetEdges(raw, None, None, ctypes.byref(n)) == 0
    src, dst = (ctypes.c_void_p * n.value)(), (ctypes.c_void_p * n.value)()
    assert pw._lib.hipGraphGetEdges(raw, src, dst, ctypes.byref(n)) == 0
    return len(set(src)) < n.value


def _check_fork(L, cfg, T, eager_fork):
    """One chain and two, call by call and captured, give the same bits; only
    the capture with two chains has branches."""
    import torch
    from paper_2607_16184_amd.layer import PagedLayer
    n = cfg.n_shared
    L.set_shared_experts(n)
    plan = Plan(cfg.E, cfg.K + n, cfg.H, cfg.F, T, n_shared=n, pages=L.stats()[0])
    assert plan.fork_shared == eager_fork and (plan.fork_shared_graph if n else plan.fork_chains)
    logits, x = to_dev(synth.logits(cfg)), to_dev16(synth.activations(cfg))
    gate = to_dev(synth.shared_gate(cfg)) if n else None
    rbuf = PagedLayer.routing_buffers(T, cfg.E, cfg.K + n)
    y = torch.empty((T, cfg.H), dtype=torch.float32, device="cuda")

    def step(out):
        L.forward(x, L.route_shared(logits, cfg.K, n, gate=gate, out=rbuf), out_fp32=True, y=out)

    L.set_chains(1)
    step(y)
    torch.cuda.synchronize()
    want = y.clone()
    assert bool(torch.isfinite(want).all())
    other = torch.empty_like(y)
    for chains in (1, 2):
        L.set_chains(chains)
        y.fill_(float("nan"))
        step(y)
        torch.cuda.synchronize()
        assert torch.equal(y, want), chains
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=side):
            step(y)
        assert _branches(g) == (chains == 2), chains
        for r in range(3):
            y.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want), (chains, r)
            step(other)                                    # eager work in between
            torch.cuda.synchronize()
            assert torch.equal(other, want), (chains, r)
    return plan


@pytest.mark.parametrize("T,mtb", [(16, 1), (64, 2), (130, 4)])
def test_forked_chains_bit_identical(T, mtb):
    """The second expert chain under capture, at one, two and four slot tiles per
    pass, in a layer of 256 MiB of 16-, 8- and 4-bit pages."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], H=2048, F=5120, G=128, T=T, act=synth.BF16, sdt=synth.BF16)
    say("forked chains, T=%d" % T)
    L = gpu_random_layer(cfg)
    assert L.stats()[0] >= 256 << 20
    p = _check_fork(L, cfg, T, False)
    assert p.routed.path == DECODE and p.routed.mtb == mtb
    L.close()


@pytest.mark.parametrize("T,E,n_shared,F,eager_fork,paths", [
    (40, 10, 2, 2048, False, (DECODE, DECODE)),
    (100, 10, 2, 2048, True, (DECODE, STREAM)),
    (300, 10, 2, 2048, True, (STREAM, STREAM)),
    (600, 12, 4, 4096, True, (TILED, TILED)),
])
def test_forked_shared_experts_bit_identical(T, E, n_shared, F, eager_fork, paths):
    """The shared experts' launches on the layer's stream, on each GEMM kernel and
    with pages of 16, 8 and 4 bits; call by call where the batch is large enough."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny_shared"], E=E, n_shared=n_shared, H=1024, F=F, G=128, T=T,
                              act=synth.BF16, sdt=synth.BF16)
    say("forked shared experts, T=%d" % T)
    L = gpu_random_layer(cfg)
    p = _check_fork(L, cfg, T, eager_fork)
    assert (p.routed.path, p.shared.path) == paths
    L.close()
