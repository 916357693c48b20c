"""The exact bf16 sum where its exponent window opens, holds, fails and moves:
values at the window's edges, zeros, outliers above and below it, data with no
common window, blocks of data of different scales in a row, subnormals, the
largest values, infinities and NaNs.  Small grids, so that every wavefront
takes many chunks; every vectors-per-step instance; the result is the oracle's
correctly rounded sum bit for bit."""
import math

import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

IDENT = {"fn": "identity"}
N = 64 * 8 * 4 * 150 + 5  # 150 chunks of one 64-thread block at 4 vectors per lane, and a tail


def scaled(g, e_lo, e_hi, n=N):
    """Signed values with exponents uniform in [e_lo, e_hi] and random fractions."""
    e = torch.randint(e_lo, e_hi + 1, (n,), generator=g).double()
    m = 1.0 + torch.randint(0, 128, (n,), generator=g).double() / 128
    s = torch.randint(0, 2, (n,), generator=g).double() * 2 - 1
    return (s * m * 2.0 ** e).to(torch.float32).to(torch.bfloat16)


def normal(g, n=N):
    return torch.randn(n, generator=g).to(torch.bfloat16)


def patch(x, where, value):
    x = x.clone()
    x[where] = value
    return x


def datasets(g):
    x = normal(g)
    yield "normal", x
    yield "relu", torch.relu(x)
    yield "zeros", torch.zeros(N, dtype=torch.bfloat16)
    yield "zeros_then_normal", torch.cat([torch.zeros(N // 2, dtype=torch.bfloat16), x[: N - N // 2]])
    yield "negative_zero", torch.full((N,), -0.0, dtype=torch.bfloat16)
    # the first vectors hold 2^0: the window is [2^-35, 2^5)
    one = patch(x.clamp(-1.5, 1.5), slice(0, 2048), 1.0)
    yield "window_top", patch(one, slice(3000, N, 97), 31.875)
    yield "above_top", patch(one, slice(3000, N, 9973), -32.0)
    yield "window_bottom", patch(one, slice(3000, N, 97), 2.0 ** -35)
    yield "below_bottom", patch(one, slice(3000, N, 9973), 2.0 ** -36 * 1.9921875)
    yield "no_window", scaled(g, -60, 60)
    yield "whole_range", scaled(g, -126, 126)
    yield "scales_in_a_row", torch.cat([scaled(g, 20 * k - 100, 20 * k - 90, N // 10 + 1) for k in range(10)])[:N]
    yield "subnormal", scaled(g, -133, -120)
    yield "largest", scaled(g, 105, 127)
    yield "large_edge", scaled(g, 104, 107)  # largest + 4 exponents: the last window and none
    yield "one_sign", patch(scaled(g, -2, 4).abs(), slice(0, 5), 2.0 ** -30)
    yield "inf", patch(x, 40000, math.inf)
    yield "both_inf", patch(patch(x, 40000, math.inf), 7, -math.inf)
    yield "nan", patch(x, N - 1, math.nan)


@pytest.mark.parametrize("unroll", [1, 2, 4])
def test_exact_bf16_windows(unroll):
    dev = torch.device("cuda", 0)
    op, dt, a = hdc.OP_TRANSFORM_REDUCE, hdc.BF16, hdc.ACC_EXACT
    saved = {b: hdc.get_tuning(op, dt, a, b) for b in range(hdc.BUCKETS)}
    g = torch.Generator().manual_seed(230904000 + unroll)
    ws = torch.empty(hdc.workspace_size(op, dt, a, N), dtype=torch.uint8, device=dev)
    try:
        for name, x in datasets(g):
            xg = x.to(dev)
            ref = oracle.reduce(IDENT, x)["exact"]
            for block, gm in ((64, 1), (256, 8)):
                hdc.set_tuning(op, dt, a, -1, block=block, unroll=unroll, grid_mult=gm)
                # 6 views: one block's grid shrinks to a few by the size, alignment of head and tail varies
                for lo, n in ((0, N), (0, 2048 * 7), (3, 5000), (1, 9)):
                    want = ref if (lo, n) == (0, N) else oracle.reduce(IDENT, x[lo:lo + n])["exact"]
                    print(f"exact window {name} unroll={unroll} block={block} gm={gm} lo={lo} n={n}", flush=True)
                    got = hdc.transform_reduce(xg[lo:lo + n], IDENT, "exact", ws=ws).item()
                    assert got == want or (math.isnan(got) and math.isnan(want)), (name, block, lo, n, got, want)
    finally:
        for b, t in saved.items():
            hdc.set_tuning(op, dt, a, b, **t)


def test_exact_bf16_many_chunks_per_lane():
    """One 64-thread block per CU over data whose lanes take the most vectors the launch allows."""
    dev = torch.device("cuda", 0)
    op, dt, a = hdc.OP_TRANSFORM_REDUCE, hdc.BF16, hdc.ACC_EXACT
    n = (1 << 25) + 8 * 77 + 3
    saved = hdc.get_tuning(op, dt, a, 3)
    gd = torch.Generator(device=dev).manual_seed(230904010)
    x = torch.randn(n, generator=gd, device=dev).abs().to(torch.bfloat16)
    x[5::100003] = 2.0 ** -100
    x[1 << 23:: 1 << 20] = 2.0 ** 90
    ref = oracle.reduce(IDENT, x.cpu())["exact"]
    try:
        for block, unroll, gm in ((64, 4, 1), (64, 1, 1), (512, 4, 4)):
            hdc.set_tuning(op, dt, a, 3, block=block, unroll=unroll, grid_mult=gm)
            print(f"exact window many chunks block={block} unroll={unroll}", flush=True)
            assert hdc.transform_reduce(x, IDENT, "exact").item() == ref
    finally:
        hdc.set_tuning(op, dt, a, 3, **saved)
