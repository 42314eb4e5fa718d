"""The matrix-core router against the oracle, bit for bit: every workgroup
shape its rule picks, ragged token and expert blocks, one to many stages,
logits that depend on the order and the rounding of their sums, masked
experts, and the kernels that take over for operands that are not 16-byte
aligned."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2410_12247_amd import moe, synth
from tests.gpu_util import bf16, dev, f32, off_by

gpu = pytest.mark.gpu


def draw(T, E, H, use_bias, seed):
    rng = np.random.default_rng(seed)
    xb = synth.bf16_bits(rng.standard_normal((T, H), dtype=np.float32))
    wr = rng.standard_normal((E, H), dtype=np.float32) * np.float32(0.05)
    bias = rng.standard_normal(E, dtype=np.float32) * np.float32(0.1) if use_bias else None
    return xb, wr, bias


def check(x, w_router, bias, want_ids, want_w, T, E, H, k, renorm):
    d = moe.dims(T, H, 64, E, k, renormalize=renorm)
    ids = torch.full((T, k), -1, dtype=torch.int32, device=dev())
    w = torch.full((T, k), -1.0, dtype=torch.float32, device=dev())
    moe.route(d, x, w_router, bias, ids, w)
    torch.cuda.synchronize()
    assert np.array_equal(ids.cpu().numpy(), want_ids)
    # the fp64 softmax rounds once to fp32: at most one unit in the last place
    np.testing.assert_array_max_ulp(w.cpu().numpy(), want_w, maxulp=1)


def shape(T, E):
    """(tokens of a workgroup, expert blocks per wave) of the fused kernel for
    more than 16 experts, as the library picks it (256 compute units without a
    device, the MI355X's count)."""
    fn = moe.lib().moe_router_shape_for_tests
    blocks = ctypes.c_int32()
    tok = fn(ctypes.byref(moe.dims(T, 64, 64, E, 1)), ctypes.byref(blocks))
    return tok, blocks.value


# one ragged (tokens, experts) per workgroup shape on 256 compute units
SHAPES = {
    (16, 1): (41, 49), (16, 2): (1003, 113), (16, 3): (3001, 161), (16, 4): (300, 250),
    (32, 1): (5, 17), (32, 2): (4203, 64), (32, 3): (8189, 90), (32, 4): (4999, 128),
    (32, 5): (6007, 145), (32, 6): (4150, 192), (32, 8): (8001, 230),
    (64, 1): (8237, 31), (64, 2): (8240, 33), (64, 3): (9001, 96), (64, 4): (12330, 97),
    (64, 5): (8193, 160), (64, 6): (12345, 177), (64, 8): (16383, 193),
    (128, 1): (16411, 29), (128, 2): (24585, 50), (128, 3): (24600, 81), (128, 4): (24999, 120),
    (128, 5): (32767, 160), (128, 6): (24601, 170), (128, 8): (28733, 256),
}


def test_shapes_cover_the_rule():
    """SHAPES names every shape the rule picks, each under its own key."""
    if torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("written for 256 compute units")
    seen = {shape(T, E) for E in range(17, 257, 8) for T in list(range(1, 40000, 97)) + [65536]}
    assert seen == set(SHAPES)
    for want, (T, E) in SHAPES.items():
        assert shape(T, E) == want, (want, T, E)


@gpu
@pytest.mark.parametrize("want", list(SHAPES))
def test_every_shape(want):
    """Ragged token and expert blocks, five stages (rings of two and three),
    bias and full softmax."""
    T, E = SHAPES[want]
    H, k = 320, 3
    xb, wr, bias = draw(T, E, H, True, T + E)
    _, ids, w = oracle.route(xb, wr, bias, k, False)
    check(bf16(xb), f32(wr), f32(bias), ids, w, T, E, H, k, False)


def order_sensitive(T, E, H, seed):
    """Operands whose logits depend on the order and the rounding of the sum:
    terms of magnitude 2^-8 to 2^16 that cancel, products of 32 significant
    bits, and for three experts in four denormal products only."""
    rng = np.random.default_rng(seed)
    xb = synth.bf16_bits(rng.choice([-1.0, 1.0], (T, H)).astype(np.float32) *
                         (1 + rng.integers(0, 128, (T, H)).astype(np.float32) / 128))
    wr = (rng.choice([-1.0, 1.0], (E, H)) * np.exp2(rng.integers(-8, 17, (E, H))) *
          (1 + rng.integers(0, 1 << 23, (E, H)) / (1 << 23))).astype(np.float32)
    # the second half of h takes the first half's terms away again: what is
    # left are the roundings
    wr[:, H // 2:] = -wr[:, :H // 2]
    xb[:, H // 2:] = xb[:, :H // 2]
    tiny = np.arange(E) % 4 != 0
    wr[tiny] = (rng.integers(-64, 65, wr[tiny].shape) * 2.0 ** -149).astype(np.float32)
    return xb, wr, tiny


def pairwise_logits(xb, wr):
    """The same products in groups of four added pairwise, in fp32."""
    x = synth.bf16_to_f32(xb)
    z = np.zeros((len(x), len(wr)), np.float32)
    for h in range(0, x.shape[1], 4):
        p = x[:, None, h:h + 4] * wr[None, :, h:h + 4]
        z += (p[..., 0] + p[..., 1]) + (p[..., 2] + p[..., 3])
    return z


@gpu
@pytest.mark.parametrize("T,E,off,call", [
    (40, 16, 0, "route"),            # a chain per lane
    (600, 8, 0, "route"),            # matrix cores, at most 16 experts
    (600, 8, 1, "route"),            # a lane per token
    (97, 40, 0, "route"),            # matrix cores, selection in the workgroup
    (97, 40, 1, "route"),            # register tiles
    (97, 40, 0, "forward"),          # matrix cores, a selection launch
    (97, 40, 1, "forward"),          # a lane per token, a selection launch
])
def test_sums_in_order(T, E, off, call):
    """Every logit is one fma chain over ascending h with denormals kept: with
    these operands another order picks other experts."""
    H, k = 192, 8
    xb, wr, tiny = order_sensitive(T, E, H, 3 * T + E)
    z, ids, w = oracle.route(xb, wr, None, k, False)
    other = np.argsort(-pairwise_logits(xb, wr), axis=1, kind="stable")[:, :k]
    assert (other != ids).any(axis=1).mean() > 0.5, "the operands have to tell the orders apart"
    flushed = np.argsort(-np.where(tiny, 0, z), axis=1, kind="stable")[:, :k]
    assert (flushed != ids).any(axis=1).mean() > 0.5, "... and denormals from zero"
    if call == "route":
        check(off_by(bf16(xb), off), f32(wr), None, ids, w, T, E, H, k, False)
        return
    d = moe.dims(T, H, 64, E, k, 0, 1, False)
    g = torch.zeros((1, 64, H), dtype=torch.bfloat16, device=dev())
    buf = moe.MoEBuffers(d, moe.opts())
    buf.run(off_by(bf16(xb), off), f32(wr), None, g, g, g.view(1, H, 64))
    torch.cuda.synchronize()
    assert np.array_equal(buf.topk_ids.cpu().numpy(), ids)
    np.testing.assert_array_max_ulp(buf.topk_w.cpu().numpy(), w, maxulp=1)


@gpu
@pytest.mark.parametrize("T,E,H,k,renorm,use_bias", [
    (513, 8, 64, 2, True, False),       # E <= 16: one wave per workgroup, one stage
    (4095, 16, 320, 8, False, True),    # its last full block, stages not a multiple of the ring
    (4097, 13, 128, 3, True, True),     # four waves
    (1, 17, 64, 8, True, False),        # one token, a block of one expert
    (33, 33, 192, 2, False, True),      # 16 tokens x 4 waves of 1 block of experts
    (4097, 64, 64, 8, True, False),     # 32 tokens x 2 waves of 2
    (8193, 160, 128, 6, False, True),   # 64 tokens x 2 waves of 5
    (33000, 160, 64, 6, True, False),   # 32 tokens x 2 waves of 5
    (9000, 208, 64, 5, True, True),     # 16 tokens x 4 waves of 4, 13 blocks
    (300, 256, 448, 8, False, False),   # the most experts
])
def test_shapes(T, E, H, k, renorm, use_bias):
    xb, wr, bias = draw(T, E, H, use_bias, 31 * T + E)
    _, ids, w = oracle.route(xb, wr, bias, k, renorm)
    check(bf16(xb), f32(wr), f32(bias) if use_bias else None, ids, w, T, E, H, k, renorm)


@gpu
@pytest.mark.parametrize("T,E", [(5, 8), (700, 8), (600, 160)])
def test_masked_experts(T, E):
    """Experts masked by a bias of -inf or the lowest float are never chosen
    and weigh nothing in the full softmax."""
    xb, wr, bias = draw(T, E, 128, True, T + E)
    bias[1::4] = -np.inf
    bias[2::4] = np.finfo(np.float32).min
    _, ids, w = oracle.route(xb, wr, bias, 3, False)
    check(bf16(xb), f32(wr), f32(bias), ids, w, T, E, 128, 3, False)


@gpu
@pytest.mark.parametrize("T,E,k,call", [(5, 8, 8, "route"), (700, 8, 8, "route"),
                                         (3, 20, 6, "route"), (600, 160, 8, "route"),
                                         (70, 256, 8, "forward"), (2, 40, 8, "forward")])
def test_nan_logits_pick_distinct_experts(T, E, k, call):
    """NaN logits have no defined weights, but a token's experts stay distinct:
    the finite ones first, then the NaNs of all one bits (the lowest key there
    is) by index.  A repeated expert would exceed the row bounds that the
    dispatch buffers and the GEMM tiles are sized by."""
    H = 128
    xb, wr, bias = draw(T, E, H, True, T + E)
    finite = [1, E // 2, E - 1]
    b = np.full(E, 0xFFFFFFFF, np.uint32)
    b[finite] = bias[finite].view(np.uint32)
    bias = b.view(np.float32)
    d = moe.dims(T, H, 64, E, k, E - 3, 3, renormalize=False)
    if call == "route":
        ids = torch.full((T, k), -1, dtype=torch.int32, device=dev())
        moe.route(d, bf16(xb), f32(wr), f32(bias), ids,
                  torch.empty((T, k), dtype=torch.float32, device=dev()))
        counts = None
    else:
        w = torch.zeros((3, 64, H), dtype=torch.bfloat16, device=dev())
        buf = moe.MoEBuffers(d, moe.opts())
        buf.run(bf16(xb), f32(wr), f32(bias), w, w, w.view(3, H, 64))
        ids, counts = buf.topk_ids, buf.counts.cpu().numpy()
    torch.cuda.synchronize()
    ids = ids.cpu().numpy()
    assert np.array_equal(np.sort(ids[:, :3], axis=1), np.tile(sorted(finite), (T, 1)))
    rest = [e for e in range(E) if e not in finite][:k - 3]
    assert np.array_equal(ids[:, 3:], np.tile(rest, (T, 1)))
    if counts is not None:
        assert counts.max() <= T and counts.tolist() == [
            int((ids == e).sum()) for e in range(E - 3, E)]


@gpu
@pytest.mark.parametrize("T,E,off", [
    (600, 40, 4), (600, 160, 4),  # x eight bytes off: one token per thread, 3 and 32 x 5 experts
    (600, 100, 2),                # 8 experts per thread
    (16385, 30, 1),               # two tokens and 2 experts per thread
    (16384, 250, 1),              # two tokens and 16 experts per thread
    (65537, 64, 1),               # four tokens and 4 experts per thread
    (65536, 160, 1),              # four tokens and 10 experts per thread
])
def test_unaligned_rows(T, E, off):
    """x off a 16-byte boundary, more than 16 experts, no logits buffer: the
    register-tiled kernel."""
    H, k = 192 if T < 1000 else 64, 4
    xb, wr, bias = draw(T, E, H, True, E)
    _, ids, w = oracle.route(xb, wr, bias, k, True)
    check(off_by(bf16(xb), off), f32(wr), f32(bias), ids, w, T, E, H, k, True)


@gpu
@pytest.mark.parametrize("T,E,xoff", [
    (3, 8, 0), (40, 16, 0),            # a chain per lane
    (600, 8, 0), (5000, 16, 0),        # matrix cores, at most 16 experts
    (33, 40, 0), (4097, 160, 0),       # matrix cores, more experts
    (100, 8, 1), (600, 160, 1),        # x unaligned too: lane per token, register tiles
])
def test_unaligned_router(T, E, xoff):
    """w_router four bytes off a 16-byte boundary."""
    H, k = 320, 4
    xb, wr, bias = draw(T, E, H, True, T + E)
    _, ids, w = oracle.route(xb, wr, bias, k, True)
    check(off_by(bf16(xb), xoff), off_by(f32(wr), 1), f32(bias), ids, w, T, E, H, k, True)


@gpu
@pytest.mark.parametrize("T", [4, 61])
def test_unaligned_router_in_the_forward(T):
    """The same with the logits through the workspace and, at four tokens, the
    dispatch behind the selection."""
    E, H, k = 40, 320, 4
    xb, wr, bias = draw(T, E, H, True, T)
    _, ids, w = oracle.route(xb, wr, bias, k, True)
    z = torch.zeros((E, 64, H), dtype=torch.bfloat16, device=dev())
    buf = moe.MoEBuffers(moe.dims(T, H, 64, E, k, renormalize=True), moe.opts())
    buf.run(bf16(xb), off_by(f32(wr), 1), f32(bias), z, z, z.view(E, H, 64))
    torch.cuda.synchronize()
    assert np.array_equal(buf.topk_ids.cpu().numpy(), ids)
    np.testing.assert_array_max_ulp(buf.topk_w.cpu().numpy(), w, maxulp=1)
    assert np.array_equal(buf.counts.cpu().numpy(), np.bincount(ids.ravel(), minlength=E))


@gpu
@pytest.mark.parametrize("E", [8, 16, 17, 160])
@pytest.mark.parametrize("T", [1, 3, 4, 5])
def test_dispatch_behind_the_router(T, E):
    """A router launch of one workgroup also computes the dispatch indices;
    with every phase timed they take a launch of their own.  The same bits,
    whole and in expert or token stages, and the row counts of the ids."""
    H, I, k = 128, 64, 8
    xb, wr, bias = draw(T, E, H, True, 7 * T + E)
    rng = np.random.default_rng(E)
    w = lambda *s: bf16(synth.bf16_bits(  # noqa: E731
        rng.standard_normal(s, dtype=np.float32) * np.float32(0.05)))
    e0, EL = (1, 6) if E < 100 else (30, 100)
    wg, wu, wd = w(EL, I, H), w(EL, I, H), w(EL, H, I)
    d = moe.dims(T, H, I, E, k, e0, EL, True)
    for stage in ({}, {"pipeline_n": 2}, {"pipeline_n": 2, "chunk_mode": moe.CHUNK_TOKENS}):
        if stage.get("chunk_mode") is not None and (T < 2 or 2 * EL > 256):
            continue
        out = []
        for timing in (False, True):
            b = moe.MoEBuffers(d, moe.opts(timing=timing, exact_order=True, **stage))
            b.run(bf16(xb), f32(wr), f32(bias), wg, wu, wd)
            torch.cuda.synchronize()
            out.append((b.y.cpu(), b.topk_ids.cpu(), b.topk_w.cpu(), b.counts.cpu()))
        for a, c in zip(*out):
            assert torch.equal(a, c)
        ids = out[0][1].numpy().ravel() - e0
        want = np.bincount(ids[(ids >= 0) & (ids < EL)], minlength=EL)
        assert np.array_equal(out[0][3].numpy(), want)
