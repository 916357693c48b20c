"""Long runs of empty segments in the tiled segmented reduce: at the start, in
the middle of a tile, at a tile's edge and at the end of the range, of 62 to
300,000 segments (a batch of offsets holds 64), and a range with no element at
all, in the pass with the scan (one launch and two) and in the pass without
it.  Results against the oracle, and the time of a call: no part of it may
grow by a dependent read per segment of a run."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
HOR, IDENT = {"fn": "horner", "coef": synth.horner_coefficients(8)}, {"fn": "identity"}
IAFF = {"fn": "affine", "a": 3, "b": -7}
CLASSES = [(torch.float32, "plain", HOR), (torch.bfloat16, "compensated", IDENT), (torch.int32, "exact_int", IAFF)]
# mean length of the segments with elements, elements: one launch; two with the scan; two without it
SHAPES = {"one_launch": (40, 60_000), "two_scan": (40, 6_000_000), "two_split": (2000, 12_000_000)}


def lengths(mean, n, run):
    rng = np.random.default_rng(230905100)
    L = rng.integers(1, 2 * mean, max(8, n // mean))
    k = len(L) // 3
    edge = np.array([4096 - int(L[:k].sum()) % 4096])  # the run behind it begins at a tile's edge
    zeros = np.zeros(run, dtype=np.int64)
    return np.concatenate([zeros, L[:k], edge, zeros, L[k:2 * k], zeros, L[2 * k:], zeros])


def run_once(x, off, fn, acc, total=None):
    code, a, S = hdc.DTYPE[x.dtype], hdc.ACC[acc], off.numel() - 1
    size = hdc.workspace_size(hdc.OP_SEGMENTED_REDUCE, code, a, x.numel() if total is None else total, S)
    ws = torch.full((max(size, 256),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.full((S,), 77, dtype=hdc.OUT_DTYPE[a], device="cuda")
    return out, lambda: hdc.segmented_reduce(x, off, fn, acc, out=out, ws=ws)


@pytest.mark.parametrize("run", [62, 63, 64, 65, 127, 5000, 300_000])
@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=["f32", "bf16", "i32"])
def test_runs(dt, acc, fn, shape, run):
    off = synth.offsets_from_lengths(torch.as_tensor(lengths(*SHAPES[shape], run)))
    n = int(off[-1])
    if dt == torch.int32:
        x = synth.uniform_int(230905101, 0, n, bits=20)
    else:
        x = synth.to_storage(synth.uniform_pm1_f32(230905101, 0, n).double(), dt)
    ref = oracle.segmented(fn, x, off)
    out, call = run_once(x.cuda(), off.cuda(), fn, acc)
    print(f"empty runs {dt} {shape} run={run}", flush=True)
    for _ in range(2):
        call()
    got = out.cpu().numpy()
    if acc == "exact_int":
        assert np.array_equal(got, ref["isum"])
    else:
        assert np.all(np.abs(got - ref["exact"]) <= TOL * ref["abs_sum"])


@pytest.mark.parametrize("segments", [1, 2000, 5000, 3_000_000])
def test_no_element(segments):
    x = torch.empty(0, dtype=torch.float32, device="cuda")
    off = torch.full((segments + 1,), 0, dtype=torch.int64, device="cuda")
    out, call = run_once(x, off, IDENT, "plain")
    call()
    assert torch.count_nonzero(out).item() == 0


@pytest.mark.parametrize("shape", list(SHAPES) + ["no_element"])
def test_time_of_a_long_run(shape):
    """Four runs of 500,000 empty segments take less than 1 ms (16 MB of offsets and 8 MB of zeros; the call
    itself takes under 0.1 ms), where one dependent read per segment or per 64 of them takes 4 ms or more."""
    run = 500_000
    if shape == "no_element":
        off = torch.zeros(4 * run + 1, dtype=torch.int64)
    else:
        off = synth.offsets_from_lengths(torch.as_tensor(lengths(*SHAPES[shape], run)))
    x = torch.rand(int(off[-1]), device="cuda")
    out, call = run_once(x, off.cuda(), HOR, "plain")
    call()
    times = []
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    print(f"empty runs {shape}: {min(times):.3f} ms", flush=True)
    assert min(times) < 1.0
