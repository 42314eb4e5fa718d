"""The matrix-core router against the oracle, bit for bit: every workgroup
shape its rule picks, ragged token and expert blocks, one to many stages,
masked experts, and the kernels that take over for operands that are not
16-byte aligned."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_2410_12247_amd import moe, synth
from tests.gpu_util import bf16, dev, f32, off_by

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("T,E,H,k,renorm,use_bias", [
    (513, 8, 64, 2, True, False),       # E <= 16: one wave per workgroup, one stage
    (4095, 16, 320, 8, False, True),    # its last full block, stages not a multiple of the ring
    (4097, 13, 128, 3, True, True),     # four waves
    (1, 17, 64, 8, True, False),        # one token, a block of one expert
    (33, 33, 192, 2, False, True),      # 16 tokens x 4 waves of experts
    (4097, 64, 64, 8, True, False),     # 32 tokens
    (8193, 160, 128, 6, False, True),   # 64 tokens, a ragged last workgroup
    (33000, 160, 64, 6, True, False),   # 128 tokens
    (9000, 208, 64, 5, True, True),     # 13 blocks of experts in two waves of 8
    (300, 256, 448, 8, False, False),   # the most experts
])
def test_shapes(T, E, H, k, renorm, use_bias):
    xb, wr, bias = draw(T, E, H, use_bias, 31 * T + E)
    _, ids, w = oracle.route(xb, wr, bias, k, renorm)
    check(bf16(xb), f32(wr), f32(bias) if use_bias else None, ids, w, T, E, H, k, renorm)


@pytest.mark.parametrize("T,E", [(5, 8), (700, 8), (600, 160)])
def test_masked_experts(T, E):
    """Experts masked by a bias of -inf or the lowest float are never chosen
    and weigh nothing in the full softmax."""
    xb, wr, bias = draw(T, E, 128, True, T + E)
    bias[1::4] = -np.inf
    bias[2::4] = np.finfo(np.float32).min
    _, ids, w = oracle.route(xb, wr, bias, 3, False)
    check(bf16(xb), f32(wr), f32(bias), ids, w, T, E, 128, 3, False)


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
