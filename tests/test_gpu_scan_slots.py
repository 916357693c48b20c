"""Single-pass scans of one tile, of the few tiles whose look-back nodes lie in
library memory, and of the first tile count that goes back to the workspace:
tile counts 1, 2, 64, 65, 255, 256, 257 with ragged ends, plain and segmented,
from a workspace filled with ones, in rows of calls of changing size and type
on one workspace (earlier nodes must never count), and in a replayed graph with
eager calls in between.  Integers bit-exact against the oracle, and the status
word 0 after every call."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

IDENT = {"fn": "identity"}
HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}
TILE = 64 * 16
COUNTS = [1, 2, 64, 65, 255, 256, 257]
CLASSES = [(torch.int32, "exact_int", IDENT), (torch.float32, "plain", HOR), (torch.bfloat16, "compensated", IDENT)]


def gpu():
    return torch.device("cuda", 0)


@pytest.fixture(autouse=True)
def small_tiles():
    keys = [(hdc.DTYPE[dt], hdc.ACC[acc], b) for dt, acc, _ in CLASSES for b in range(hdc.BUCKETS)]
    saved = {k: hdc.get_tuning(hdc.OP_SCAN, *k) for k in keys}
    for dt, acc, _ in CLASSES:
        hdc.set_tuning(hdc.OP_SCAN, hdc.DTYPE[dt], hdc.ACC[acc], -1, block=64, unroll=4)
    yield
    for k, t in saved.items():
        hdc.set_tuning(hdc.OP_SCAN, *k, **t)


def make(n, dt):
    if dt == torch.int32:
        return synth.uniform_int(230904600, 0, n, bits=20)
    return synth.to_storage(synth.uniform_pm1_f32(230904600, 0, n).double(), dt)


def check(y, ref, dt, what):
    if dt == torch.int32:
        assert np.array_equal(y.cpu().numpy(), ref["isum"]), what
    else:
        assert np.all(np.abs(y.cpu().double().numpy() - ref["exact"]) <= 1e-6 * ref["abs_sum"]), what


@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=["i32", "f32", "bf16"])
def test_tile_counts(dt, acc, fn):
    x = make(COUNTS[-1] * TILE, dt)
    xg = x.to(gpu())
    ws = torch.empty(hdc.workspace_size(hdc.OP_SCAN, hdc.DTYPE[dt], hdc.ACC[acc], x.numel()), dtype=torch.uint8,
                     device=gpu())
    for tiles in COUNTS:
        n = tiles * TILE - 5
        off = torch.tensor([0, 7, 7, n // 3, n - 1, n], dtype=torch.int64)
        ref, sref = oracle.scan(fn, x[:n], True), oracle.segmented_scan(fn, x[:n], off, False)
        ws.fill_(0xFF)
        for rep in range(3):
            print(f"scan slots {dt} tiles={tiles} rep={rep}", flush=True)
            check(hdc.scan(xg[:n], fn, acc, True, ws=ws), ref, dt, (tiles, rep))
            check(hdc.segmented_scan(xg[:n], off.to(gpu()), fn, acc, False, ws=ws), sref, dt, (tiles, rep))
            assert hdc.scan_status(ws) == 0


def test_changing_sizes_on_one_workspace():
    xs = {dt: make(300 * TILE, dt).to(gpu()) for dt, _, _ in CLASSES}
    ws = torch.empty(hdc.workspace_size(hdc.OP_SCAN, hdc.I32, hdc.ACC_EXACT_INT, 300 * TILE), dtype=torch.uint8,
                     device=gpu())
    for k in range(150):
        dt, acc, fn = CLASSES[k % 3]
        n = 1 + (7919 * k * k) % (300 * TILE)
        y = hdc.scan(xs[dt][:n], fn, acc, ws=ws, check=False)
        if dt == torch.int32:
            assert torch.equal(y, torch.cumsum(xs[dt][:n].long(), 0)), (k, n)
        else:  # against the three-pass schedule
            code, a, b = hdc.DTYPE[dt], hdc.ACC[acc], hdc.tuning_bucket(n)
            hdc.set_tuning(hdc.OP_SCAN, code, a, b, unroll=1)
            z = hdc.scan(xs[dt][:n], fn, acc, ws=ws, check=False)
            hdc.set_tuning(hdc.OP_SCAN, code, a, b, unroll=4)
            assert torch.allclose(y.double(), z.double(), rtol=1e-5, atol=1e-2), (k, n)


def test_replayed_graph():
    n = 100 * TILE + 9
    x = make(n, torch.int32).to(gpu())
    ws = torch.empty(hdc.workspace_size(hdc.OP_SCAN, hdc.I32, hdc.ACC_EXACT_INT, n), dtype=torch.uint8, device=gpu())
    y = torch.empty(n, dtype=torch.int64, device=gpu())
    want = torch.cumsum(x.long(), 0)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hdc.scan(x, IDENT, "exact_int", out=y, ws=ws, check=False)
    for _ in range(6):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and hdc.scan_status(ws) == 0
        hdc.scan(x[: n // 3], IDENT, "exact_int", ws=ws)
        torch.cuda.synchronize()
