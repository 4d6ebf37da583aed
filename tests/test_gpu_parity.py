"""GPU parity against the CPU oracle, through the C ABI.

Bit-exact: quantized codes, scales and zeros (as pool bytes), routing ids,
offsets, sorted slots and slot positions. Tolerance: routing weights 1e-6
absolute; layer output max|y - r| / max|r| <= 2e-2 for the 16-bit output
against the oracle (fp64, unrounded SwiGLU output) and <= 1e-3 for the fp32
output against the oracle with the SwiGLU output rounded to the activation
dtype (the kernel's own rounding point).
"""
import numpy as np
import pytest

import oracle
from helpers import case, gpu_layer, oracle_layer, rel_err, say, to_dev, to_dev16, y16_values
from paper_2607_16184_amd import synth

pytestmark = pytest.mark.gpu

TOL16 = 2e-2
TOL32 = 1e-3
WTOL = 1e-6


def _route_check(logits, K, renorm=1):
    import torch
    from paper_2607_16184_amd import pw
    from paper_2607_16184_amd.layer import PagedLayer
    T, E = logits.shape
    lg = to_dev(logits)
    ids = torch.empty((T, K), dtype=torch.int32, device="cuda")
    w = torch.empty((T, K), dtype=torch.float32, device="cuda")
    off = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    ss = torch.empty(max(T * K, 1), dtype=torch.int32, device="cuda")
    sp = torch.empty(max(T * K, 1), dtype=torch.int32, device="cuda")
    pw.pw_route_topk(lg.data_ptr(), T, E, K, renorm, ids.data_ptr(), w.data_ptr(), off.data_ptr(),
                     ss.data_ptr(), sp.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    oid, ow = oracle.route(logits, K, renorm)
    cnt, ooff, oss, osp = oracle.permute(oid, E)
    assert np.array_equal(ids.cpu().numpy(), oid)
    assert np.abs(w.cpu().numpy() - ow).max() <= WTOL
    assert np.array_equal(off.cpu().numpy(), ooff)
    assert np.array_equal(ss.cpu().numpy()[:T * K], oss)
    assert np.array_equal(sp.cpu().numpy()[:T * K], osp)


@pytest.mark.parametrize("name", ["tiny", "mixtral_decode", "mixtral_prefill", "finegrained"])
def test_route_bit_exact(name):
    cfg = synth.CONFIGS[name]
    say("route %s T=%d E=%d K=%d" % (name, cfg.T, cfg.E, cfg.K))
    _route_check(synth.logits(cfg), cfg.K)


def test_route_edge_cases():
    rng = np.random.default_rng(5)
    say("route edge cases")
    lg = rng.standard_normal((300, 8)).astype(np.float32)
    lg[:100, :4] = 0.25                         # ties go to the lower index
    _route_check(lg, 2)
    _route_check(lg, 8)                         # K = E
    _route_check(lg, 2, renorm=0)
    _route_check(np.zeros((5, 16), np.float32), 3)
    _route_check(rng.standard_normal((1, 64)).astype(np.float32), 6)
    _route_check(rng.standard_normal((3000, 256)).astype(np.float32), 16)   # several permute chunks
    # one wave per token (more than 32 experts): ties, +0 and -0 (equal
    # values: the lower index first), all-negative rows
    lg = -np.abs(rng.standard_normal((200, 64))).astype(np.float32) - 1.0
    lg[:50, 10:20] = 0.5
    lg[50:100, 7] = -0.0
    lg[50:100, 3] = 0.0
    lg[50:100, 40] = -0.0
    _route_check(lg, 6)
    _route_check(lg, 6, renorm=0)
    # unrenormalised weights on the one-wave-per-token path: a partly filled
    # block of 64 lanes (E = 60) and four logits per lane (E = 256)
    _route_check(rng.standard_normal((500, 60)).astype(np.float32), 4, renorm=0)
    _route_check(rng.standard_normal((500, 256)).astype(np.float32), 8, renorm=0)


def _check_pages(L, O, pages):
    for (e, p, rb) in pages:
        got = L.page_image(e, p, rb)
        want = O.page_image(p, e, rb)
        assert got.size == want.size
        if not np.array_equal(got, want):
            b = int(O.bits[p][e, rb])
            R, K = O.R, O.w16[p].shape[2]
            gc, gs, gz = oracle.decode_page(got, R, K, O.G, b)
            _, wc, ws, wz = O.page(p, e, rb)
            raise AssertionError("page %s bits %d: codes %d, scales %d, zeros %d mismatches" % (
                (e, p, rb), b, (gc != wc).sum(), (gs != ws).sum(), (gz != wz).sum()))


def test_tiny_quantized_pages_bit_exact():
    cfg, w16, bits, order = case("tiny")
    say("tiny: load %d pages" % len(order))
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    _check_pages(L, O, order)
    L.close()


# Every bitwidth pair at G = 64 (two groups per 128-value block), 128 (one)
# and 256 / 512 (a group over two or four blocks, coded in two passes), with
# fp16 and bf16 activations and scales.
@pytest.mark.parametrize("src,dst,G,act,sdt", [
    (16, 8, 64, synth.F16, synth.F16), (16, 4, 64, synth.F16, synth.F16), (8, 4, 64, synth.F16, synth.F16),
    (16, 8, 128, synth.BF16, synth.BF16), (16, 4, 128, synth.BF16, synth.BF16), (8, 4, 128, synth.BF16, synth.BF16),
    (8, 4, 128, synth.F16, synth.BF16),
    (16, 8, 256, synth.BF16, synth.F16), (16, 4, 256, synth.F16, synth.BF16), (8, 4, 256, synth.BF16, synth.BF16),
    (16, 4, 512, synth.BF16, synth.F16), (8, 4, 512, synth.F16, synth.F16),
])
def test_tiny_requant_bit_exact(src, dst, G, act, sdt):
    import torch
    extra = dict(H=512, F=1024) if G == 512 else {}
    cfg, w16, _, order = case("tiny", G=G, act=act, sdt=sdt, **extra)
    bits = [np.full((cfg.E, cfg.nrb(p)), src, np.int32) for p in range(3)]
    say("tiny requant %d->%d G=%d act=%d sdt=%d" % (src, dst, G, act, sdt))
    L = gpu_layer(cfg, w16, bits, order, slack=1.0)
    O = oracle_layer(cfg, w16, bits)
    blocks = [pg for i, pg in enumerate(order) if i % 3 == 0]
    side = torch.cuda.Stream()
    delta = L.requant(blocks, dst, stream=side)
    want = 0
    for (e, p, rb) in blocks:
        want += O.requant(p, e, rb, dst)
    assert delta == want
    assert L.commit() == len(blocks)
    torch.cuda.synchronize()
    _check_pages(L, O, order)
    assert L.reclaim() > 0
    L.close()


def test_requant_mixed_pairs_several_launches():
    """One requant call over 600 pages of a 32-expert layer, mixing the three
    bitwidth pairs (16 -> 8, 16 -> 4, 8 -> 4) and both K (gate/up and down
    pages): the 16 -> 4 pages take two launches of at most 448 pages. Every
    page of the layer is compared byte for byte afterwards."""
    import torch
    from paper_2607_16184_amd import pw
    cfg, w16, _, order = case("tiny", E=32)
    rng = np.random.default_rng(11)
    bits = [np.where(rng.random((cfg.E, cfg.nrb(p))) < 0.2, 8, 16).astype(np.int32) for p in range(3)]
    say("requant: 32-expert tiny layer, mixed pairs over %d pages" % len(order))
    L = gpu_layer(cfg, w16, bits, order, slack=1.0)
    O = oracle_layer(cfg, w16, bits)
    blocks, new = [], []
    for (e, p, rb) in order:
        b = int(bits[p][e, rb])
        nb = 4 if b == 8 else (8 if rng.random() < 0.1 else 4)
        blocks.append((e, p, rb))
        new.append(nb)
    pairs = [(int(bits[p][e, rb]), nb) for (e, p, rb), nb in zip(blocks, new)]
    assert set(pairs) == {(16, 8), (16, 4), (8, 4)}
    assert pairs.count((16, 4)) > 448          # 449 here: a second launch of one page
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    es, ps, rbs = zip(*blocks)
    delta = pw.pw_requant_blocks(L.handle, list(es), list(ps), list(rbs), new, side.cuda_stream)
    want = sum(O.requant(p, e, rb, nb) for (e, p, rb), nb in zip(blocks, new))
    assert delta == want
    assert L.commit() == len(blocks)
    torch.cuda.synchronize()
    _check_pages(L, O, order)
    assert L.reclaim() > 0
    L.close()


def _forward_parity(cfg, L, O, x16, logits, tokens=None, w_round=False):
    import torch
    routing = L.route(to_dev(logits), cfg.K)
    x = to_dev16(x16)
    y16 = L.forward(x, routing)
    y32 = L.forward(x, routing, out_fp32=True)
    torch.cuda.synchronize()
    ids, w = oracle.route(logits, cfg.K)
    r1 = O.forward(x16, ids, w, h_round=False, tokens=tokens)
    r2 = O.forward(x16, ids, w, h_round=True, tokens=tokens, w_round=w_round)
    sel = slice(None) if tokens is None else list(tokens)
    e16 = rel_err(y16_values(y16, cfg.act)[sel], r1[sel])
    e32 = rel_err(y32.cpu().numpy()[sel], r2[sel])
    return e16, e32, y16, y32


def test_tiny_forward_parity():
    cfg, w16, bits, order = case("tiny")
    say("tiny forward")
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    e16, e32, y16, y32 = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg))
    assert e16 <= TOL16, e16
    assert e32 <= TOL32, e32
    L.close()


@pytest.mark.parametrize("b", [16, 8, 4])
def test_tiny_uniform_bitwidth(b):
    """Every block at one bitwidth: the same kernel, a uniform configuration."""
    cfg, w16, _, order = case("tiny")
    bits = [np.full((cfg.E, cfg.nrb(p)), b, np.int32) for p in range(3)]
    say("tiny uniform %d" % b)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg))
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


def test_tiny_deterministic_and_pool_order_invariant():
    import torch
    cfg, w16, bits, order = case("tiny")
    say("tiny determinism / pool order")
    L1 = gpu_layer(cfg, w16, bits, order)
    L2 = gpu_layer(cfg, w16, bits, list(reversed(order)))
    x = to_dev16(synth.activations(cfg))
    r1 = L1.route(to_dev(synth.logits(cfg)), cfg.K)
    a = L1.forward(x, r1, out_fp32=True).clone()
    b = L1.forward(x, r1, out_fp32=True).clone()
    c = L2.forward(x, r1, out_fp32=True).clone()
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
    assert L1.entry(0, 0, 0).data_off != L2.entry(0, 0, 0).data_off or \
        L1.entry(cfg.E - 1, 2, 0).data_off != L2.entry(cfg.E - 1, 2, 0).data_off
    L1.close()
    L2.close()


def test_zero_up_projection_gives_zero():
    import torch
    cfg, w16, bits, order = case("tiny")
    w16 = list(w16)
    w16[1] = np.zeros_like(w16[1])
    say("tiny zero up")
    L = gpu_layer(cfg, w16, [np.full_like(b, 16) for b in bits], order)
    y = L.forward(to_dev16(synth.activations(cfg)), L.route(to_dev(synth.logits(cfg)), cfg.K), out_fp32=True)
    torch.cuda.synchronize()
    assert not y.cpu().numpy().any()
    L.close()


# Large per-expert slot counts (at least 128 expected per expert) take the
# LDS-tiled GEMM with 256-slot tiles; medium ones (49..127) take it too where its
# tiles fill the chip (tests/test_gpu_tiles.py), and in layers as small as these
# the streaming GEMM with 64-slot tiles. Both feed quantized weights to the MFMA
# as fl32(z + c*s) rounded to the activation dtype, so their fp32 output is
# compared with the oracle read the same way (w_round).

@pytest.mark.parametrize("T", [1000, 1531])
def test_tiny_tiled_path_parity(T):
    cfg, w16, bits, order = case("tiny", T=T)
    say("tiny tiled T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg), w_round=True)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


@pytest.mark.parametrize("b", [16, 8, 4])
def test_tiny_tiled_uniform_and_empty_experts(b):
    """Every page at one bitwidth; all slots on experts 0 and 1 (ragged tails
    of 1100 slots, six experts with none)."""
    cfg, w16, _, order = case("tiny", T=1100)
    bits = [np.full((cfg.E, cfg.nrb(p)), b, np.int32) for p in range(3)]
    lg = synth.logits(cfg).copy()
    lg[:, :2] += 100.0
    say("tiny tiled uniform %d, two experts" % b)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    toks = list(range(0, 1100, 7)) + [1099]
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), lg, tokens=toks, w_round=True)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


@pytest.mark.parametrize("T", [300, 211])
def test_tiny_stream_path_parity(T):
    """49..127 expected slots per expert: the streaming GEMM (64-slot tiles)."""
    cfg, w16, bits, order = case("tiny", T=T)
    say("tiny stream T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg), w_round=True)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


@pytest.mark.parametrize("b", [16, 8, 4])
def test_tiny_stream_uniform_and_empty_experts(b):
    """Every page at one bitwidth; 200 tokens all routed to experts 3 and 5
    (four 64-slot tiles each, the last ragged; six experts with none)."""
    cfg, w16, _, order = case("tiny", T=200)
    bits = [np.full((cfg.E, cfg.nrb(p)), b, np.int32) for p in range(3)]
    lg = synth.logits(cfg).copy()
    lg[:, [3, 5]] += 100.0
    say("tiny stream uniform %d, two experts" % b)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), lg, w_round=True)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


# 21..48 expected slots per expert: the decode kernels with up to four 16-slot
# tiles per pass, each wave streaming two 16-row weight tiles (exact
# code-domain arithmetic, so no w_round).
@pytest.mark.parametrize("T", [100, 190])
def test_tiny_decode4_path_parity(T):
    cfg, w16, bits, order = case("tiny", T=T)
    say("tiny decode, four slot tiles, T=%d" % T)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    toks = list(range(0, T, 3)) + [T - 1]
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg), tokens=toks)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


@pytest.mark.parametrize("b", [16, 8, 4])
def test_tiny_decode4_uniform_and_heavy_experts(b):
    """Every page at one bitwidth; 100 tokens all routed to experts 3 and 5
    (100 slots each: a 64-slot pass and a ragged 36-slot pass; six experts
    with none)."""
    cfg, w16, _, order = case("tiny", T=100)
    bits = [np.full((cfg.E, cfg.nrb(p)), b, np.int32) for p in range(3)]
    lg = synth.logits(cfg).copy()
    lg[:, [3, 5]] += 100.0
    say("tiny decode4 uniform %d, two experts" % b)
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    toks = list(range(0, 100, 3)) + [99]
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), lg, tokens=toks)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


# Group sizes above 128 (a group spans 2 or 4 128-blocks; on the decode path
# the down projection's K splits must hold whole groups) and scale/zero dtypes
# other than the activation dtype, on each of the three GEMM paths: 16 tokens
# (4 expected slots per expert) and 120 tokens (30: four slot tiles, two row
# tiles per wave; 8-wave workgroups, or 4-wave ones when H = 384 does not
# divide into 256-row down units) decode, 300 the streaming GEMM, 1000 the
# tiled.
@pytest.mark.parametrize("act,sdt,G,H,F,T", [
    (synth.BF16, synth.F16, 256, 256, 512, 16),
    (synth.F16, synth.BF16, 512, 512, 1024, 16),
    (synth.BF16, synth.F16, 128, 256, 512, 16),
    (synth.F16, synth.BF16, 128, 256, 512, 16),
    (synth.BF16, synth.F16, 256, 256, 512, 120),
    (synth.BF16, synth.BF16, 128, 384, 512, 120),
    (synth.F16, synth.BF16, 256, 256, 512, 300),
    (synth.BF16, synth.F16, 512, 512, 1024, 1000),
])
def test_tiny_group_sizes_and_scale_dtypes(act, sdt, G, H, F, T):
    cfg, w16, bits, order = case("tiny", act=act, sdt=sdt, G=G, H=H, F=F, T=T)
    say("tiny act=%d sdt=%d G=%d H=%d F=%d T=%d" % (act, sdt, G, H, F, T))
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    toks = None if T <= 16 else list(range(0, T, 9)) + [T - 1]
    e16, e32, _, _ = _forward_parity(cfg, L, O, synth.activations(cfg), synth.logits(cfg), tokens=toks,
                                     w_round=T > 200)
    assert e16 <= TOL16 and e32 <= TOL32, (e16, e32)
    L.close()


# Edge shapes on the decode path: a single token, every expert selected
# (K = E), unrenormalised routing weights (through the fused router at 8
# experts and the one-wave-per-token router at 64), a 64-expert top-6 layer
# with few tokens (most experts empty), and no tokens at all.
@pytest.mark.parametrize("T,K,E,renorm", [(1, 2, 8, 1), (3, 8, 8, 1), (7, 2, 8, 0), (5, 6, 64, 1),
                                          (40, 6, 64, 0)])
def test_tiny_edge_shapes(T, K, E, renorm):
    import torch
    cfg, w16, bits, order = case("tiny", T=T, K=K, E=E)
    say("tiny edge T=%d K=%d E=%d renorm=%d" % (T, K, E, renorm))
    L = gpu_layer(cfg, w16, bits, order)
    O = oracle_layer(cfg, w16, bits)
    logits, x16 = synth.logits(cfg), synth.activations(cfg)
    routing = L.route(to_dev(logits), K, renorm=renorm)
    y32 = L.forward(to_dev16(x16), routing, out_fp32=True)
    torch.cuda.synchronize()
    ids, w = oracle.route(logits, K, renorm)
    assert np.array_equal(routing[0].cpu().numpy(), ids)
    r2 = O.forward(x16, ids, w, h_round=True)
    assert rel_err(y32.cpu().numpy(), r2) <= TOL32
    L.close()


def test_zero_tokens():
    import torch
    cfg, w16, bits, order = case("tiny")
    say("tiny, no tokens")
    L = gpu_layer(cfg, w16, bits, order)
    logits = torch.zeros((0, cfg.E), dtype=torch.float32, device="cuda")
    x = torch.zeros((0, cfg.H), dtype=torch.int16, device="cuda")
    routing = L.route(logits, cfg.K)
    y = L.forward(x, routing, out_fp32=True)
    torch.cuda.synchronize()
    assert tuple(y.shape) == (0, cfg.H)
    assert not routing[2].cpu().numpy().any()      # every expert offset is 0
    L.close()
