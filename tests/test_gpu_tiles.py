"""Edges of the tiled and the streaming paged GEMM: expert slot counts around
the tile widths, every group layout (scale/zero groups of 64, 128, 256 values in
4- and 8-bit units), short reductions and mixed page formats, against the CPU
oracle. (F = 8192 gives 4 experts a gate/up tile for every CU, which the tiled
kernel needs below 128 slots per expert.)

The kernels multiply quantized weights rounded to the activation dtype
(w_round) and round the SwiGLU output there too; what is left between the
two is the order of fp32 sums over K <= 8192 products (about sqrt(K) 2^-24,
5e-6), far below the 1e-3 allowed (the bound the other fp32 parity tests use). The decode kernels'
two-row-tile form (layers with few 16-bit pages) keeps weights exact, so it
is held to the same bound against the plain oracle.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from helpers import gpu_layer, gpu_random_layer, oracle_layer, rel_err, say, to_dev, to_dev16
from paper_2607_16184_amd import synth
from test_gemm_plan import DECODE, STREAM, TILED, Plan

pytestmark = pytest.mark.gpu

F16, BF16 = synth.F16, synth.BF16


@pytest.mark.parametrize("counts,H,F,R,G,act,sdt", [
    ((1, 127, 128, 129), 256, 256, 64, 64, F16, F16),       # streaming, 64-slot tiles: one slot, ragged, full, one over
    ((63, 0, 250, 65), 256, 384, 64, 128, BF16, BF16),      # streaming: an empty expert, four tiles
    ((1, 127, 128, 129), 256, 8192, 64, 64, F16, F16),      # 128-slot tiles, one slot, full, one over
    ((63, 0, 250, 65), 256, 8192, 64, 128, BF16, BF16),     # an empty expert, two tiles
    ((64, 49, 17, 90), 512, 8192, 128, 256, F16, BF16),     # groups over two 128-blocks
    ((255, 256, 257, 0), 512, 256, 128, 256, BF16, F16),    # 256-slot tiles
    ((500, 16, 17, 15), 256, 640, 64, 64, BF16, BF16),      # skew: idle waves in most tiles
    ((300, 129, 240, 1), 768, 128, 128, 128, F16, BF16),    # K = 128: one block per row of the down pages
    ((100, 90, 70, 120), 384, 256, 64, 64, BF16, BF16),     # H not a multiple of 256: the streaming kernel
    (tuple(37 * e % 101 for e in range(130)), 256, 256, 64, 64, BF16, BF16),   # the tile search passes 64 experts twice
])
def test_tile_edges(counts, H, F, R, G, act, sdt):
    import torch
    E, T = len(counts), sum(counts)
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], E=E, K=1, H=H, F=F, R=R, G=min(G, H, F), T=T, act=act, sdt=sdt)
    w16 = [synth.expert_weights(cfg, p) for p in range(3)]
    bits = synth.bitmap(cfg)
    say("tiles %s H=%d F=%d G=%d act=%d" % (counts, H, F, cfg.G, act))
    L = gpu_layer(cfg, w16, bits, synth.pool_order(cfg))
    O = oracle_layer(cfg, w16, bits)
    lg = synth.logits(cfg).copy()
    own = np.random.default_rng(3).permutation(np.repeat(np.arange(E), counts))
    lg[np.arange(T), own] += 100.0
    x16 = synth.activations(cfg)
    y = L.forward(to_dev16(x16), L.route(to_dev(lg), 1), out_fp32=True)
    torch.cuda.synchronize()
    ids, w = oracle.route(lg, 1)
    assert np.array_equal(np.bincount(ids[:, 0], minlength=E), counts)
    e = rel_err(y.cpu().numpy(), O.forward(x16, ids, w, h_round=True, w_round=True))
    assert e <= 1e-3, e
    L.close()


@pytest.mark.parametrize("T,share16,H,G,act,sdt", [
    (16, 0.0, 256, 64, F16, F16),        # one slot tile per pass
    (60, 0.12, 256, 128, BF16, BF16),    # two, an eighth of the pages at 16 bits
    (33, 0.0, 512, 256, BF16, F16),      # groups over two 128-blocks
    (16, 0.0, 384, 128, F16, BF16),      # an odd number of 128-blocks
])
def test_decode_two_row_tiles(T, share16, H, G, act, sdt):
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], H=H, F=2048, R=64, G=G, T=T, act=act, sdt=sdt,
                              mix=(share16, 0.4, 0.6 - share16))
    w16 = [synth.expert_weights(cfg, p) for p in range(3)]
    bits = synth.bitmap(cfg)
    say("two row tiles T=%d H=%d G=%d act=%d" % (T, H, G, act))
    L = gpu_layer(cfg, w16, bits, synth.pool_order(cfg))
    O = oracle_layer(cfg, w16, bits)
    lg, x16 = synth.logits(cfg), synth.activations(cfg)
    y = L.forward(to_dev16(x16), L.route(to_dev(lg), cfg.K), out_fp32=True)
    torch.cuda.synchronize()
    ids, w = oracle.route(lg, cfg.K)
    e = rel_err(y.cpu().numpy(), O.forward(x16, ids, w, h_round=True))
    assert e <= 1e-3, e
    L.close()


@pytest.mark.parametrize("T,G", [(16, 128), (60, 64), (33, 256)])
def test_row_tiles_give_the_same_bits(T, G):
    """One or two row tiles per wave: two layers that differ only in the bitwidth
    of the pages of two experts that no token uses (4, then 16 bits: a quarter
    of the pages) run the two forms on the same pages."""
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], H=1024, F=2048, R=64, G=G, T=T, act=BF16, sdt=BF16)
    lg = synth.logits(cfg).copy()
    lg[:, 6:] -= 100.0
    x, out = to_dev16(synth.activations(cfg)), []
    for unused in (4, 16):
        say("row tiles T=%d G=%d, unused pages at %d bits" % (T, G, unused))
        bits = [np.array([[unused if e >= 6 else (8, 4)[(e + rb) % 2] for rb in range(cfg.nrb(p))]
                          for e in range(cfg.E)], np.int32) for p in range(3)]
        L = gpu_random_layer(cfg, bits=bits)
        out.append(L.forward(x, L.route(to_dev(lg), cfg.K), out_fp32=True))
        torch.cuda.synchronize()
        L.close()
    assert torch.equal(out[0], out[1])


def test_narrow_tiles_keep_within_static_workspace():
    """100 slots per expert, 3200 slots of H = 4096: the SwiGLU rows and one copy
    of the down partials fit the allocation-free entry point's 64 MiB, two
    copies would not, so the call is taken with one and gives the same bits as
    with a workspace of the caller's. (32 gate/up tiles: the streaming kernel;
    test_split_follows_the_workspace has the tiled one.)"""
    import torch
    from paper_2607_16184_amd import pw
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], E=32, K=1, H=4096, F=128, T=3200, act=BF16, sdt=BF16)
    say("narrow tiles in the static workspace")
    L = gpu_layer(cfg, [synth.expert_weights(cfg, p) for p in range(3)], synth.bitmap(cfg), synth.pool_order(cfg))
    one = cfg.T * (cfg.F * 2 + cfg.H * 4)
    assert one <= 64 << 20 < one + cfg.T * cfg.H * 4
    assert pw.pw_workspace_bytes(L.handle, cfg.T, 1) <= 64 << 20
    x = to_dev16(synth.activations(cfg))
    routing = L.route(to_dev(synth.logits(cfg)), 1)
    want = L.forward(x, routing, out_fp32=True)
    y = torch.full_like(want, float("nan"))
    _, w, off, ss, sp = routing
    pw.pw_moe_paged_gemm_noalloc(L.handle, x.data_ptr(), cfg.T, 1, w.data_ptr(), off.data_ptr(), ss.data_ptr(),
                                 sp.data_ptr(), y.data_ptr(), 1, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    L.close()


def test_split_follows_the_workspace():
    """120 slots per expert over 128 experts: the plan splits the down projection
    in two, which takes more than the static 64 MiB. With a workspace for one
    copy of the partials, and through the allocation-free entry point, the call
    runs unsplit with the same bits; with one byte less it is refused. The
    split sums the same products in another order (F = 1280: relative 1e-5)."""
    import torch
    from paper_2607_16184_amd import pw
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], E=128, K=1, H=256, F=1280, T=15360, act=BF16, sdt=BF16)
    say("split by the workspace, 128 experts")
    L = gpu_random_layer(cfg)
    one = cfg.T * (cfg.F * 2 + cfg.H * 4)
    full = pw.pw_workspace_bytes(L.handle, cfg.T, 1)
    assert one <= 64 << 20 < full == one + cfg.T * cfg.H * 4
    x = to_dev16(synth.activations(cfg))
    routing = L.route(to_dev(synth.logits(cfg)), 1)
    split = L.forward(x, routing, out_fp32=True)
    _, w, off, ss, sp = routing
    ptrs = (w.data_ptr(), off.data_ptr(), ss.data_ptr(), sp.data_ptr())
    st = torch.cuda.current_stream().cuda_stream
    ws = torch.empty(one + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    small, static = torch.full_like(split, float("nan")), torch.full_like(split, float("nan"))
    pw.pw_moe_paged_gemm(L.handle, x.data_ptr(), cfg.T, 1, *ptrs, small.data_ptr(), 1, base, one, st)
    pw.pw_moe_paged_gemm_noalloc(L.handle, x.data_ptr(), cfg.T, 1, *ptrs, static.data_ptr(), 1, st)
    with pytest.raises(pw.PWError) as ei:
        pw.pw_moe_paged_gemm(L.handle, x.data_ptr(), cfg.T, 1, *ptrs, small.data_ptr(), 1, base, one - 1, st)
    assert ei.value.status == pw.PW_ENOMEM
    torch.cuda.synchronize()
    assert torch.equal(small, static)
    assert rel_err(small.cpu().numpy(), split.cpu().numpy()) <= 1e-5
    L.close()


# Gates of the SwiGLU test: the linear part of the sigmoid, its tails, where
# exp(-g) and 1 + exp(-g) leave the normal range, and beyond it.
GATES = [0.0, 1e-20, -1e-20, 0.01, -0.01, 0.7, -0.7, 2.5, -2.5, 5.0, -5.0, 12.0, -12.0, 20.0, -20.0, 40.0, -40.0, 60.0, -60.0,
         80.0, -80.0, 86.5, -86.5, 87.5, -87.5, 88.5, -88.5, 89.5, -89.5, 95.0, -95.0, 300.0, -300.0, 1e30, -1e30,
         float("inf"), float("-inf"), float("nan")]


@pytest.mark.parametrize("T,F,path", [(40, 512, DECODE), (60, 512, DECODE), (130, 512, DECODE), (240, 512, STREAM),
                                      (240, 8192, TILED), (600, 512, TILED)])
def test_swiglu_rows_by_element(T, F, path):
    """The SwiGLU rows element by element over given gates, on every GEMM path
    (the tiled one with either tile). Column 0 of x times 4 is the gate (twice
    the largest bf16 makes it infinite) and column 1 the up value, through
    16-bit pages that are zero elsewhere, so both reach SwiGLU exact (a NaN
    gate comes with a NaN up). silu(g) u in fp32 is within a few 2^-24 of the
    value and is then rounded to bf16: at most one step apart, 2^-7 of the
    value, and 1 / (1 + exp(-g)) may vanish where it is below 2^-126."""
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], E=4, K=1, F=F, T=T, act=BF16, sdt=BF16)
    assert Plan(4, 1, cfg.H, F, T).routed.path == path
    say("swiglu rows T=%d F=%d" % (T, F))
    w = [np.zeros((4, F, 256), np.float32), np.zeros((4, F, 256), np.float32), np.zeros((4, 256, F), np.float32)]
    w[0][:, :, 0] = 4.0
    w[1][:, :, 1] = np.array([1.0, -0.75])[np.arange(F) % 2]
    bits = [np.full((4, cfg.nrb(p)), 16, np.int32) for p in range(3)]
    L = gpu_layer(cfg, [synth.to16(v, BF16) for v in w], bits, synth.pool_order(cfg))
    x = np.zeros((T, 256), np.float32)
    g = np.array([GATES[t % len(GATES)] for t in range(T)], np.float32)
    x[:, 0] = np.where(np.isinf(g), np.sign(g) * np.float32(3e38), g / 4)
    x[:, 1] = np.array([1.0, -3.0, 0.125])[np.arange(T) // len(GATES) % 3]
    x16 = synth.to16(x, BF16)
    lg = np.zeros((T, 4), np.float32)
    lg[np.arange(T), np.arange(T) % 4] = 100.0
    routing = L.route(to_dev(lg), 1)
    L.forward(to_dev16(x16), routing, out_fp32=True)
    torch.cuda.synchronize()
    rows = L.hidden_rows(T, 1).cpu().numpy().view(np.uint16)
    got = np.empty((T, F), np.float64)
    got[routing[3].cpu().numpy()] = synth.from16(rows, BF16)
    xs = synth.from16(x16, BF16)
    with np.errstate(all="ignore"):
        gate = (xs[:, 0] * np.float32(4)).astype(np.float64)[:, None]          # overflows in fp32 as in the kernels
        up = xs[:, 1].astype(np.float64)[:, None] * w[1][0, :, 1].astype(np.float64) + 0.0 * xs[:, :1]
        want = gate / (1.0 + np.exp(-gate)) * up
        want[(gate < -89.0)[:, 0] & np.isfinite(gate)[:, 0]] = 0.0             # exp(-g) is infinite in fp32
        bad, inf = np.isnan(want), np.isinf(want)
        assert bad.any() and inf.any()
        assert np.array_equal(np.isnan(got), bad)
        assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
        wrong = np.abs(got - want) > 2.0 ** -7 * np.abs(want) + 90.0 * 2.0 ** -126 * np.abs(up)
        assert not wrong[~inf].any(), gate[wrong.any(axis=1), 0]
    L.close()


def test_swiglu_over_the_exponent_range():
    """Gate values of a few hundred either way: exp(-g) overflows, vanishes and
    passes through everything between; the output keeps the usual bound."""
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], K=1, T=600, act=BF16, sdt=BF16)
    w16 = [synth.expert_weights(cfg, p) for p in range(3)]
    bits = synth.bitmap(cfg)
    say("swiglu over the exponent range")
    L = gpu_layer(cfg, w16, bits, synth.pool_order(cfg))
    O = oracle_layer(cfg, w16, bits)
    lg = synth.logits(cfg)
    x16 = synth.to16(300.0 * synth.from16(synth.activations(cfg), BF16), BF16)   # g ~ N(0, 96)
    y = L.forward(to_dev16(x16), L.route(to_dev(lg), 1), out_fp32=True)
    torch.cuda.synchronize()
    ids, w = oracle.route(lg, 1)
    got = y.cpu().numpy()
    assert np.isfinite(got).all()
    e = rel_err(got, O.forward(x16, ids, w, h_round=True, w_round=True))
    assert e <= 1e-3, e
    L.close()


@pytest.mark.parametrize("act", [F16, BF16])
@pytest.mark.parametrize("T", [16, 60, 130])
def test_activation_sums_by_half_blocks(T, act):
    """The decode kernels' activation sums X add 64-value half blocks on their own
    before they meet: 2^15 and -2^15 in the second half leave nothing of
    themselves in the sum of small values of the first (one running fp32 sum
    would cut those to multiples of 2^-8, X by up to 2^-9). Gate and up pages of
    ones (every group: scale 0, zero 1) make both projections X, so the SwiGLU
    rows are silu(X) X: two roundings to 16 bits apart at most, and 64
    roundings to fp32 inside X."""
    import torch
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], E=4, K=1, R=64, G=128, T=T, act=act, sdt=act)
    say("activation sums T=%d act=%d" % (T, act))
    ones = np.full((4, cfg.F, cfg.H), synth.to16(np.ones(1, np.float32), act)[0])
    bits = [np.array([[(8, 4)[rb % 2] for rb in range(cfg.nrb(p))]] * 4, np.int32) for p in range(3)]
    L = gpu_layer(cfg, [ones, ones, synth.expert_weights(cfg, 2)], bits, synth.pool_order(cfg))
    x = np.zeros((T, cfg.H), np.float32)
    x[:, :64] = 0.125 * np.random.default_rng(7).standard_normal((T, 64))
    x[:, 70], x[:, 100] = 32768.0, -32768.0
    x16 = synth.to16(x, act)
    routing = L.route(to_dev(synth.logits(cfg)), 1)
    L.forward(to_dev16(x16), routing, out_fp32=True)
    torch.cuda.synchronize()
    got = np.empty((T, cfg.F))
    got[routing[3].cpu().numpy()] = synth.from16(L.hidden_rows(T, 1).cpu().numpy().view(np.uint16), act)
    X = synth.from16(x16, act).astype(np.float64).sum(1)
    want = (X * X / (1.0 + np.exp(-X)))[:, None]
    assert (got == got[:, :1]).all()
    ulp, dx = (2.0 ** -10 if act == F16 else 2.0 ** -7), 64 * 2.0 ** -24
    assert np.all(np.abs(got - want) <= ulp * np.abs(want) + 2.0 * dx * np.abs(X)[:, None]), np.abs(got / want - 1.0).max()
    L.close()
