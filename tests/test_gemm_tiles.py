"""Tiles of the expert GEMMs at their edges: widths of one 64-column block and
of several, K of one and a few stages, row counts around the 16-row
fragments and the tile heights, and workgroups that walk many tiles (each
tile's first stages are requested before the previous tile's outputs are
written)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2410_12247_amd import moe
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu

ROWS = [0, 1, 15, 16, 17, 63, 65, 127, 128, 129, 191, 193, 255, 257, 319, 321, 640]


def ints(rng, *shape):
    return torch.from_numpy(rng.integers(-2, 3, shape).astype(np.float32)).to(dev(), torch.bfloat16)


def reference(x, wg, wu, wd):
    """y in 64 bits and a bound on the error of a correct result: the sums of
    these integers are exact in fp32, the activation is rounded to bf16 (half
    an ulp, 2^-9, plus the hardware exp2 and reciprocal) and the down sum adds
    its own fp32 roundings."""
    g, u = x.double() @ wg.double().t(), x.double() @ wu.double().t()
    act = g * torch.sigmoid(g) * u
    bound = (act.abs() @ wd.double().abs().t()) * 2.0 ** -8 + 1e-6
    return act @ wd.double().t(), bound


@pytest.mark.parametrize("H,I,cu_budget", [
    (64, 64, 8),      # one stage (or two), one partial column tile; 8 workgroups
    (128, 192, 8),    # gate/up: a full and a partial column tile
    (320, 128, 16),   # down: a full and a partial column tile
    (576, 448, 0),    # odd stage counts, one tile per workgroup
])
def test_group_tiles(H, I, cu_budget):
    rng = np.random.default_rng(H + I)
    E, R = len(ROWS), sum(ROWS)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(ROWS)]).astype(np.int32)).to(dev())
    x = ints(rng, R, H)
    wg, wu, wd = ints(rng, E, I, H), ints(rng, E, I, H), ints(rng, E, H, I)
    d = moe.dims(R, H, I, E, 1, renormalize=True)
    act = torch.zeros((R, I), dtype=torch.bfloat16, device=dev())
    y = torch.full((R + 1, H), 7.0, device=dev())
    moe.ffn_group(d, 0, E, off, x, wg, wu, wd, act, y[:R], cu_budget)
    torch.cuda.synchronize()
    assert bool((y[R] == 7.0).all()), "wrote past the last row"
    for e in range(E):
        r0, r1 = int(off[e]), int(off[e + 1])
        want, bound = reference(x[r0:r1], wg[e], wu[e], wd[e])
        assert bool(((y[r0:r1].double() - want).abs() <= bound).all()), f"expert of {ROWS[e]} rows"


@pytest.mark.parametrize("rows", [1, 16, 127, 129, 321, 1000])
@pytest.mark.parametrize("H,I", [(64, 64), (320, 192)])
def test_dense_tiles(rows, H, I):
    rng = np.random.default_rng(rows + H)
    x, wg, wu, wd = ints(rng, rows, H), ints(rng, I, H), ints(rng, I, H), ints(rng, H, I)
    act = torch.zeros((rows, I), dtype=torch.bfloat16, device=dev())
    y = torch.full((rows + 1, H), 7.0, device=dev())
    moe.ffn_dense(rows, H, I, x, wg, wu, wd, act, y[:rows])
    torch.cuda.synchronize()
    assert bool((y[rows] == 7.0).all()), "wrote past the last row"
    want, bound = reference(x, wg, wu, wd)
    assert bool(((y[:rows].double() - want).abs() <= bound).all())


@pytest.mark.parametrize("I", [64, 128, 1024])
@pytest.mark.parametrize("rows", [
    [0, 1, 16, 17, 32, 33, 64],
    [0, 1, 2, 15, 16, 17, 32],  # at most 32: three workgroups resident per compute unit
])
def test_skinny_heights_mixed(rows, I):
    """One decode launch whose experts have 0 to 64 rows: each expert's rows
    pick the height of its down tiles; K of fewer stages than the ring and of
    more."""
    H, E, R = 4736, len(rows), sum(rows)  # 7 x 74 tiles: two to three per compute unit
    rng = np.random.default_rng(5)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).to(dev())
    x = ints(rng, R, H)
    wg, wu, wd = ints(rng, E, I, H), ints(rng, E, I, H), ints(rng, E, H, I)
    d = moe.dims(max(rows), H, I, 8, 8, 0, E, True)
    act = torch.zeros((R, I), dtype=torch.bfloat16, device=dev())
    y = torch.full((R + 1, H), 7.0, device=dev())
    moe.ffn_group(d, 0, E, off, x, wg, wu, wd, act, y[:R])
    torch.cuda.synchronize()
    assert bool((y[R] == 7.0).all()), "wrote past the last row"
    for e in range(E):
        r0, r1 = int(off[e]), int(off[e + 1])
        want, bound = reference(x[r0:r1], wg[e], wu[e], wd[e])
        assert bool(((y[r0:r1].double() - want).abs() <= bound).all()), f"expert of {rows[e]} rows"


@pytest.mark.parametrize("T", [1, 2, 7, 16])
@pytest.mark.parametrize("H,I", [
    (64, 64),       # two K steps: most waves have none
    (320, 192),     # ten and six steps over eight waves
    (1344, 576),    # uneven pieces, more steps than are in flight
    (576, 2112),    # the deep ring of the down GEMM
    (2304, 64),     # gate/up: nine steps per wave, eight in flight
    (4096, 128),    # sixteen
    (256, 3584),    # down: fourteen steps per wave, twelve in flight
])
def test_stream_gemms(T, H, I):
    """The forward of a few tokens without shared experts: both GEMMs stream
    the weights with K cut over the waves.  Against 64-bit sums, repeated
    calls and the no-allocation entry point bit for bit, and within the K
    split's rounding of exact order."""
    E, k, e0, EL = 8, 2, 1, 6
    rng = np.random.default_rng(T + H)
    x = torch.from_numpy(rng.standard_normal((T, H)).astype(np.float32)).to(dev(), torch.bfloat16)
    wr = torch.from_numpy(rng.standard_normal((E, H)).astype(np.float32) * 0.05).to(dev())
    w = lambda *s: torch.from_numpy(  # noqa: E731
        rng.standard_normal(s).astype(np.float32) * 0.05).to(dev(), torch.bfloat16)
    wg, wu, wd = w(EL, I, H), w(EL, I, H), w(EL, H, I)
    d = moe.dims(T, H, I, E, k, e0, EL, True)
    out = []
    for o in (moe.opts(), moe.opts(), moe.opts(exact_order=True)):
        b = moe.MoEBuffers(d, o)
        out.append((b, b.run(x, wr, None, wg, wu, wd)))
    y2 = torch.empty_like(out[0][1])
    moe.forward_noalloc(d, moe.opts(), x, wr, None, wg, wu, wd, None, None, None, y2, None, None,
                        None)
    torch.cuda.synchronize()
    b, y = out[0]
    assert torch.equal(y, out[1][1]) and torch.equal(y, y2)
    want, bound = torch.zeros(T, H, dtype=torch.float64, device=dev()), 0.0
    for t in range(T):
        for j in range(k):
            e = int(b.topk_ids[t, j]) - e0
            if 0 <= e < EL:
                r, bd = reference(x[t:t + 1], wg[e], wu[e], wd[e])
                want[t] += float(b.topk_w[t, j]) * r[0]
                bound = max(bound, float(bd.max()))
    # bf16 activations (reference's bound), doubled for the fp32 sums of
    # non-integers, over at most k experts
    assert float((y.double() - want).abs().max()) <= 2 * k * bound
    scale = float(want.abs().max())
    assert float((y - out[2][1]).abs().max()) <= 2e-2 * scale
