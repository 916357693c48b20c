"""Operands that lie differently within 16 bytes: views that start 0, 1, 3 and
7 elements into their buffers, through every entry point that streams more
than one array, at sizes around a vector, a tile and the map's size rule.
Maps and integers bit-exact, sums and prefixes within the oracle's bar, and
nothing written outside the output view."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}
FAFF = {"fn": "affine", "a": 2.5, "b": 0.5}
IAFF = {"fn": "affine", "a": 3, "b": -7}
IDENT, PROD = {"fn": "identity"}, {"fn": "product"}
DTYPES = [torch.float32, torch.float16, torch.bfloat16, torch.int32]
PAIRS = [(0, 1), (1, 0), (3, 2), (7, 4)]  # starts of the two operands
SIZES = [1, 7, 9, 17, 4099, 65535, 65536, 65551, 300007]
GUARD = 8


def gpu():
    return torch.device("cuda", 0)


def bits(t):
    return t.view({2: torch.int16, 4: torch.int32, 8: torch.int64}[t.element_size()])


def make(n, dt, seed, stream=0):
    if dt == torch.int32:
        return synth.uniform_int(seed, stream, n, bits=20)
    return synth.to_storage(synth.uniform_pm1_f32(seed, stream, n).double(), dt)


def view(x, start):
    """x on the GPU as a view that starts `start` elements into a larger buffer."""
    buf = torch.zeros(x.numel() + start + GUARD, dtype=x.dtype, device=gpu())
    buf[start:start + x.numel()] = x.to(gpu())
    return buf[start:start + x.numel()]


def output(n, dt, start):
    """An output view with the buffer around it, which must keep its fill."""
    buf = torch.full((n + start + GUARD,), 77, dtype=dt, device=gpu())
    return buf, buf[start:start + n]


def untouched(buf, start, n):
    return bool((buf[:start] == 77).all()) and bool((buf[start + n:] == 77).all())


def sum_ok(got, ref, acc, what):
    if acc == "exact_int":
        assert got == ref["isum"], what
    elif acc == "exact":
        assert got == ref["exact"], what
    else:
        assert abs(got - ref["exact"]) <= TOL * ref["abs_sum"], what


@pytest.mark.parametrize("dt", DTYPES)
def test_map_and_map_reduce(dt):
    ints = dt == torch.int32
    fm, fr, acc = (IAFF, IDENT, "exact_int") if ints else (HOR, FAFF, "compensated")
    for n in SIZES:
        x = make(n, dt, 230904100 + n)
        want, ref = oracle.map(fm, x), oracle.reduce(fr, x)
        for xs, ys in PAIRS:
            print(f"misaligned map {dt} n={n} x+{xs} y+{ys}", flush=True)
            xg = view(x, xs)
            buf, y = output(n, dt, ys)
            hdc.map(xg, fm, out=y)
            buf2, y2 = output(n, dt, ys)
            _, r = hdc.map_reduce(xg, fm, fr, acc, out=y2)
            torch.cuda.synchronize()
            assert torch.equal(bits(y.cpu()), bits(want)) and untouched(buf, ys, n), (n, xs, ys)
            assert torch.equal(bits(y2.cpu()), bits(want)) and untouched(buf2, ys, n), (n, xs, ys)
            sum_ok(r.item(), ref, acc, (n, xs, ys))


@pytest.mark.parametrize("dt,acc", [(torch.float32, "plain"), (torch.bfloat16, "compensated"),
                                    (torch.float16, "compensated"), (torch.float16, "exact")])
def test_dot(dt, acc):
    saved = {b: hdc.get_tuning(hdc.OP_DOT, hdc.DTYPE[dt], hdc.ACC[acc], b) for b in range(hdc.BUCKETS)}
    try:
        for n in SIZES:
            x, z = make(n, dt, 230904200 + n), make(n, dt, 230904200 + n, 1)
            ref = oracle.reduce(PROD, x, z)
            for xs, zs in PAIRS + [(2, 0)]:
                xg, zg = view(x, xs), view(z, zs)
                for unroll in (1, 2, 4):
                    hdc.set_tuning(hdc.OP_DOT, hdc.DTYPE[dt], hdc.ACC[acc], -1, unroll=unroll)
                    print(f"misaligned dot {dt} {acc} n={n} x+{xs} z+{zs} unroll={unroll}", flush=True)
                    sum_ok(hdc.transform_reduce(xg, PROD, acc, z=zg).item(), ref, acc, (n, xs, zs, unroll))
    finally:
        for b, t in saved.items():
            hdc.set_tuning(hdc.OP_DOT, hdc.DTYPE[dt], hdc.ACC[acc], b, **t)


def test_exact_dot_non_finite_past_the_end():
    """Values after the end of z, and an infinity in its last vector: only what belongs to the dot counts."""
    for n in (9, 4099, 65551):
        x, z = make(n, torch.float16, 230904250), make(n, torch.float16, 230904251)
        zbuf = torch.full((n + 1 + 64,), float("nan"), dtype=torch.float16, device=gpu())
        zbuf[1:1 + n] = z.to(gpu())
        assert hdc.transform_reduce(view(x, 0), PROD, "exact", z=zbuf[1:1 + n]).item() == \
            oracle.reduce(PROD, x, z)["exact"]
        zbuf[n] = float("inf")
        x[-1] = 1.0
        assert hdc.transform_reduce(view(x, 0), PROD, "exact", z=zbuf[1:1 + n]).item() == float("inf")


@pytest.mark.parametrize("dt", DTYPES)
def test_batch(dt):
    ints = dt == torch.int32
    fm, fr, acc = (IAFF, IDENT, "exact_int") if ints else (FAFF, HOR, "compensated")
    xs = [make(n, dt, 230904300 + n) for n in SIZES]
    starts = [PAIRS[i % len(PAIRS)] for i in range(len(xs))]
    bufs, ys = zip(*[output(x.numel(), dt, b) for x, (_, b) in zip(xs, starts)])
    _, outs = hdc.batch_map_reduce([view(x, a) for x, (a, _) in zip(xs, starts)], fm, fr, acc, ys=list(ys))
    torch.cuda.synchronize()
    for i, x in enumerate(xs):
        assert torch.equal(bits(ys[i].cpu()), bits(oracle.map(fm, x))), i
        assert untouched(bufs[i], starts[i][1], x.numel()), i
        sum_ok(outs[i].item(), oracle.reduce(fr, x), acc, i)


@pytest.mark.parametrize("dt,acc", [(torch.float32, "plain"), (torch.float16, "compensated"),
                                    (torch.bfloat16, "plain"), (torch.int32, "exact_int")])
def test_scans(dt, acc):
    fn = IAFF if dt == torch.int32 else HOR
    out_dt = hdc.OUT_DTYPE[hdc.ACC[acc]]
    code, a = hdc.DTYPE[dt], hdc.ACC[acc]
    saved = {b: hdc.get_tuning(hdc.OP_SCAN, code, a, b) for b in range(hdc.BUCKETS)}
    try:
        for unroll in (4, 1):  # one pass, three passes
            hdc.set_tuning(hdc.OP_SCAN, code, a, -1, unroll=unroll)
            for n in (1, 17, 4099, 65551):
                x = make(n, dt, 230904400 + n)
                off = torch.tensor([0, min(3, n), min(3, n), min(1000, n), n], dtype=torch.int64)
                ref = oracle.scan(fn, x, True)
                sref = oracle.segmented_scan(fn, x, off, False)
                for xs, ys in PAIRS + [(2, 0)]:
                    print(f"misaligned scan {dt} n={n} x+{xs} y+{ys} unroll={unroll}", flush=True)
                    buf, y = output(n, out_dt, ys)
                    buf2, y2 = output(n, out_dt, ys)
                    hdc.scan(view(x, xs), fn, acc, True, out=y)
                    hdc.segmented_scan(view(x, xs), off.to(gpu()), fn, acc, False, out=y2)
                    assert untouched(buf, ys, n) and untouched(buf2, ys, n)
                    for got, r in ((y, ref), (y2, sref)):
                        if dt == torch.int32:
                            assert np.array_equal(got.cpu().numpy(), r["isum"]), (n, xs, ys)
                        else:
                            err = np.abs(got.cpu().double().numpy() - r["exact"])
                            assert np.all(err <= TOL * r["abs_sum"]), (n, xs, ys)
    finally:
        for b, t in saved.items():
            hdc.set_tuning(hdc.OP_SCAN, code, a, b, **t)
