"""The forms of the tiled segmented reduce around their limits: the pass with
the scan in two launches (short segments, more tiles than one block folds),
exactly as many tiles as one block folds and one more or less, and a workspace
sized for exactly the elements.  Every storage type and fold, plain and
compensated, against the oracle, twice with the same bits from a workspace
filled with ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
BLOCK, CHUNK = 64, 1024
LAST = BLOCK * 4  # tiles that one block of 64 folds
HOR, IDENT = {"fn": "horner", "coef": synth.horner_coefficients(8)}, {"fn": "identity"}
IAFF = {"fn": "affine", "a": 3, "b": -7}
CLASSES = [(dt, acc, HOR) for dt in (torch.float32, torch.float16, torch.bfloat16) for acc in ("plain", "compensated")]
CLASSES += [(torch.float32, "plain", IDENT), (torch.bfloat16, "compensated", IDENT), (torch.int32, "exact_int", IAFF),
            (torch.int32, "exact_int", IDENT)]


def short(rng, n):
    """Segments of 0..60 elements that cover n, with runs of empty ones at tiles' edges."""
    L, at = [], 0
    while at < n:
        k = min(int(rng.integers(0, 61)), n - at)
        if at // CHUNK != (at + k) // CHUNK:
            k = CHUNK - at % CHUNK  # a segment that ends at the tile's edge, then empty ones
            k = min(k, n - at)
            L += [k] + [0] * int(rng.integers(0, 130))
        else:
            L.append(k)
        at += k
    return L


def layouts():
    rng = np.random.default_rng(230905600)
    yield "two_launches", short(rng, 460_000)
    yield "two_launches_ones", [1] * 330_000
    yield "two_launches_across", list(rng.integers(200, 380, 1500)) + [0] * 300 + [5000, 1, 0, 2] * 20
    for tiles in (LAST - 2, LAST - 1, LAST):  # the launcher counts two more than the whole ones
        yield f"{tiles}_tiles", short(rng, tiles * CHUNK - 1)
        yield f"{tiles}_tiles_and_a_rest", short(rng, tiles * CHUNK + 7)


@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=[f"{str(c[0])[6:]}_{c[1]}_{c[2]['fn']}" for c in CLASSES])
def test_forms(dt, acc, fn):
    op, code, a = hdc.OP_SEGMENTED_REDUCE, hdc.DTYPE[dt], hdc.ACC[acc]
    saved = {b: hdc.get_tuning(op, code, a, b) for b in range(hdc.BUCKETS)}
    try:
        hdc.set_tuning(op, code, a, -1, block=BLOCK, unroll=1, chunk=CHUNK, grid_mult=64, passes=1)
        for name, L in layouts():
            for start, shift in ((0, 0), (5, 1)):
                off = synth.offsets_from_lengths(torch.as_tensor(np.asarray(L), dtype=torch.int64)) + start
                n, S = int(off[-1]), off.numel() - 1
                if dt == torch.int32:
                    base = synth.uniform_int(230905601, 0, n + shift, bits=20)
                else:
                    base = synth.to_storage(synth.normal_f64(230905601, 0, n + shift), dt)
                ref = oracle.segmented(fn, base[shift:], off)
                xg, og = base.cuda()[shift:], off.cuda()
                ws = torch.empty(hdc.workspace_size(op, code, a, n, S), dtype=torch.uint8, device="cuda")
                got = []
                for rep in range(2):
                    ws.fill_(0xFF)
                    print(f"forms {name} {dt} {acc} start={start} rep={rep}", flush=True)
                    out = torch.full((S,), 77, dtype=hdc.OUT_DTYPE[a], device="cuda")
                    hdc.segmented_reduce(xg, og, fn, acc, out=out, ws=ws)
                    got.append(out.cpu().numpy())
                assert got[0].tobytes() == got[1].tobytes(), (name, start)
                if acc == "exact_int":
                    assert np.array_equal(got[0], ref["isum"]), (name, start)
                else:
                    err = np.abs(got[0].astype(np.float64) - ref["exact"])
                    assert np.all(err <= TOL * ref["abs_sum"]), (name, start)
    finally:
        for b, t in saved.items():
            hdc.set_tuning(op, code, a, b, **t)
