"""Tiles with many segment ends in the pass
without the scan (long segments on average, or a workspace sized for far more
elements): 6 to 9 ends in a tile of 1024 (crowded from 8 on), 61 to 66 in one of
8192 (from 63 on), segments that enter and leave such tiles,
end or start at their edges or run through several of them, the first and the
last tile with an unaligned head and tail, runs of empty segments among the
short ones; every storage type and fold against the oracle.  And the time of a
call with a stretch of short segments among long ones, which one wavefront must
not split end by end."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
TILE, BIG = 1024, 8192
SIZED_FOR = 80_000_000  # elements: thousands of tiles, and a long mean (8192 * 8192 keep a tile of 8192 whole)
HOR, IDENT = {"fn": "horner", "coef": synth.horner_coefficients(8)}, {"fn": "identity"}
IAFF = {"fn": "affine", "a": 3, "b": -7}
CLASSES = [(torch.float32, "plain", HOR), (torch.float32, "compensated", IDENT), (torch.bfloat16, "compensated", IDENT),
           (torch.float16, "plain", HOR), (torch.int32, "exact_int", IAFF)]


def layouts():
    rng = np.random.default_rng(230905300)
    for k in (6, 7, 8, 9):  # ends inside the second tile; the last segment leaves it, or ends at its edge
        yield f"{k}_ends", [TILE + 9] + [3] * (k - 1) + [3 * TILE]
        yield f"{k}_ends_to_the_edge", [TILE] + [3] * (k - 1) + [TILE - 3 * (k - 1), 5 * TILE]
        yield f"{k}_ends_with_empties", [TILE - 1, 1] + [0, 2] * (k // 2) + [2 * TILE + 7]
    for k in (61, 62, 63, 64, 65, 66):
        yield f"{k}_ends", [BIG + 9] + [30] * (k - 1) + [3 * BIG]
        yield f"{k}_ends_to_the_edge", [BIG] + [30] * (k - 1) + [BIG - 30 * (k - 1), 5 * BIG]
        yield f"{k}_ends_with_empties", [BIG - 1, 1] + [0, 20] * (k // 2) + [2 * BIG + 7]
    yield "ones", [1] * (6 * TILE + 5)
    yield "stretch", np.concatenate([[5 * TILE + 3], rng.integers(0, 9, 3000), [7 * TILE + 1], [2] * 700, [40 * TILE]])
    yield "stretches_at_both_ends", np.concatenate([rng.integers(1, 5, 900), [9 * TILE], rng.integers(1, 5, 900)])
    yield "long_in_the_middle", [2] * 100 + [700] + [2] * 100 + [300] * 20 + [1] * 200
    yield "empties", [2 * TILE + 5] + [1, 0, 0, 0] * 40 + [0] * 500 + [2] * 80 + [0] * 200 + [3 * TILE]


@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=[f"{str(c[0])[6:]}_{c[1]}" for c in CLASSES])
def test_crowded_tiles(dt, acc, fn):
    op, code, a = hdc.OP_SEGMENTED_REDUCE, hdc.DTYPE[dt], hdc.ACC[acc]
    saved = {b: hdc.get_tuning(op, code, a, b) for b in range(hdc.BUCKETS)}
    try:
        for name, L in layouts():
            for start, shift in ((0, 0), (5, 1), (3, 2)):
                off = synth.offsets_from_lengths(torch.as_tensor(np.asarray(L), dtype=torch.int64)) + start
                n, S = int(off[-1]) + 3, off.numel() - 1
                if dt == torch.int32:
                    base = synth.uniform_int(230905301, 0, n + shift, bits=20)
                else:
                    base = synth.to_storage(synth.normal_f64(230905301, 0, n + shift), dt)
                ref = oracle.segmented(fn, base[shift:], off)
                xg, og = base.cuda()[shift:], off.cuda()
                ws = torch.full((hdc.workspace_size(op, code, a, SIZED_FOR, S),), 0xFF, dtype=torch.uint8,
                                device="cuda")
                for block, unroll, chunk in ((64, 1, TILE), (256, 2, TILE), (512, 4, TILE), (256, 1, BIG)):
                    hdc.set_tuning(op, code, a, -1, block=block, unroll=unroll, chunk=chunk, grid_mult=64, passes=1)
                    print(f"crowded {name} {dt} {acc} start={start} shift={shift} block={block}", flush=True)
                    out = torch.full((S,), 77, dtype=hdc.OUT_DTYPE[a], device="cuda")
                    for _ in range(2):
                        hdc.segmented_reduce(xg, og, fn, acc, out=out, ws=ws)
                    got = out.cpu().numpy()
                    if acc == "exact_int":
                        assert np.array_equal(got, ref["isum"]), (name, start, block)
                    else:
                        err = np.abs(got.astype(np.float64) - ref["exact"])
                        assert np.all(err <= TOL * ref["abs_sum"]), (name, start, block)
    finally:
        for b, t in saved.items():
            hdc.set_tuning(op, code, a, b, **t)


def best_of_five(x, off, acc):
    code, a, S = hdc.DTYPE[x.dtype], hdc.ACC[acc], off.numel() - 1
    ws = torch.empty(hdc.workspace_size(hdc.OP_SEGMENTED_REDUCE, code, a, x.numel(), S), dtype=torch.uint8,
                     device="cuda")
    out = torch.empty(S, dtype=hdc.OUT_DTYPE[a], device="cuda")
    times = []
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        hdc.segmented_reduce(x, off, IDENT, acc, out=out, ws=ws)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return min(times[1:])


@pytest.mark.parametrize("dt,acc", [(torch.float32, "plain"), (torch.bfloat16, "compensated"), (torch.int32, "exact_int")])
def test_time_of_a_stretch(dt, acc):
    """60,000 segments of 4 elements among 100 of 500,000 take at most 40 us longer than the 100 alone (two chains
    of dependent reads and chunks, ~20 us; split end by end by the few wavefronts that hold them, 370 to 550 us)."""
    rng = np.random.default_rng(230905302)
    long = [500_000] * 50
    off = [synth.offsets_from_lengths(torch.as_tensor(np.concatenate([long, s, long]), dtype=torch.int64))
           for s in (rng.integers(1, 8, 60_000), np.zeros(0, dtype=np.int64))]
    x = torch.randint(0, 100, (int(off[0][-1]),), device="cuda").to(dt)
    with_stretch, without = (best_of_five(x[:int(o[-1])], o.cuda(), acc) for o in off)
    print(f"stretch {dt}: {with_stretch:.1f} us, without {without:.1f} us", flush=True)
    assert with_stretch <= without + 40
