"""The tiled segmented reduce where many segments end inside one chunk (its
segmented scan), where the wavefront changes between its three ways, and where
one launch folds the segments that span tiles.  Segments of one element (more
ends in a chunk than a batch of offsets holds), of a chunk and a tile and one
either side, runs of empty ones at the edges of chunks and tiles and at both
ends of the range, all empty, shifted starts; every storage type and fold, both
forms (a workspace sized for many more elements takes the second launch), and
values that must not leak into a neighbour."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}
IDENT, IAFF = {"fn": "identity"}, {"fn": "affine", "a": 3, "b": -7}
CLASSES = [(torch.float32, "plain", HOR), (torch.float32, "compensated", IDENT),
           (torch.bfloat16, "compensated", HOR), (torch.float16, "plain", IDENT), (torch.int32, "exact_int", IAFF)]


def gpu():
    return torch.device("cuda", 0)


def layouts():
    rng = np.random.default_rng(230904500)
    yield "ones", [1] * 5000
    yield "twos_and_empty", [2, 0] * 3000
    yield "short", rng.integers(0, 40, 4000)
    yield "empty_runs", [0] * 200 + [7, 0, 0, 0, 1] * 300 + [0] * 100 + [256] * 9 + [0] * 70
    yield "chunk_edges", [255, 1, 0, 0, 256, 257, 0, 511, 1, 512, 0, 513, 3, 253] * 40
    yield "tile_edges", [1024, 0, 1023, 0, 0, 1, 1025, 2048, 5, 0, 1019, 4096, 0, 3] * 12
    yield "bursts", np.concatenate([np.concatenate([[5000], rng.integers(0, 3, 700)]) for _ in range(6)])
    yield "one", [40001]
    yield "all_empty", [0] * 1000
    yield "two_between_empties", [0] * 300 + [1] + [0] * 300 + [9000] + [0] * 300


def check(got, ref, acc, what):
    got = got.cpu().numpy()
    if acc == "exact_int":
        assert np.array_equal(got, ref["isum"]), what
        return
    err = np.abs(got.astype(np.float64) - ref["exact"])
    bad = np.where(err > TOL * ref["abs_sum"])[0]
    assert bad.size == 0, (what, bad[:5])
    assert np.all(got[ref["abs_sum"] == 0] == 0.0), what


@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=[f"{str(c[0])[6:]}_{c[1]}" for c in CLASSES])
def test_dense_layouts(dt, acc, fn):
    code, a = hdc.DTYPE[dt], hdc.ACC[acc]
    saved = {b: hdc.get_tuning(hdc.OP_SEGMENTED_REDUCE, code, a, b) for b in range(hdc.BUCKETS)}
    try:
        for name, L in layouts():
            for start, shift in ((0, 0), (5, 1)):
                off = synth.offsets_from_lengths(torch.as_tensor(np.asarray(L), dtype=torch.int64)) + start
                n, S = int(off[-1]) + 3, off.numel() - 1
                if dt == torch.int32:
                    base = synth.uniform_int(230904501, 0, n + shift, bits=20)
                else:
                    base = synth.to_storage(synth.normal_f64(230904501, 0, n + shift), dt)
                ref = oracle.segmented(fn, base[shift:], off)
                xg, og = base.to(gpu())[shift:], off.to(gpu())
                for total in (n, 40_000_000):  # one launch; a workspace of many tiles: two
                    ws = torch.empty(hdc.workspace_size(hdc.OP_SEGMENTED_REDUCE, code, a, total, S),
                                     dtype=torch.uint8, device=gpu())
                    ws.fill_(0xFF)
                    for block, unroll, chunk in ((64, 1, 1024), (256, 2, 4096), (1024, 4, 1024)):
                        hdc.set_tuning(hdc.OP_SEGMENTED_REDUCE, code, a, -1, block=block, unroll=unroll, chunk=chunk,
                                       grid_mult=64, passes=1)
                        print(f"dense {name} {dt} {acc} start={start} shift={shift} total={total} block={block}",
                              flush=True)
                        out = torch.full((S,), 77, dtype=hdc.OUT_DTYPE[a], device=gpu())
                        for _ in range(2):
                            hdc.segmented_reduce(xg, og, fn, acc, out=out, ws=ws)
                        check(out, ref, acc, (name, start, total, block, unroll))
    finally:
        for b, t in saved.items():
            hdc.set_tuning(hdc.OP_SEGMENTED_REDUCE, code, a, b, **t)


@pytest.mark.parametrize("acc", ["plain", "compensated"])
def test_non_finite_values_stay_in_their_segment(acc):
    L = torch.tensor([3, 1, 0, 5, 200, 1, 1, 1, 300, 2] * 50, dtype=torch.int64)
    off = synth.offsets_from_lengths(L)
    x = synth.uniform_pm1_f32(230904502, 0, int(off[-1]))
    bad = [0, 3, 5, 57, 108, 250, 499]
    for k, j in enumerate(bad):
        if L[j] > 0:
            x[int(off[j]) + int(L[j]) // 2] = (float("nan"), float("inf"), -float("inf"))[k % 3]
    got = hdc.segmented_reduce(x.to(gpu()), off.to(gpu()), IDENT, acc).cpu().double()
    for j in range(L.numel()):
        want = x[int(off[j]):int(off[j + 1])].double().sum()
        if j in bad and L[j] > 0:
            assert torch.equal(torch.nan_to_num(got[j], 1.5, 2.5, 3.5), torch.nan_to_num(want, 1.5, 2.5, 3.5)), j
        else:
            assert abs(got[j] - want) <= TOL * x[int(off[j]):int(off[j + 1])].double().abs().sum(), j


def test_one_launch_in_a_replayed_graph():
    """Captured one-launch segmented reduces, replayed with eager calls on the same workspace in between."""
    rng = np.random.default_rng(230904503)
    off = synth.offsets_from_lengths(torch.as_tensor(rng.integers(0, 90, 5000), dtype=torch.int64))
    x = synth.uniform_pm1_f32(230904503, 0, int(off[-1])).to(gpu())
    og = off.to(gpu())
    ws = torch.empty(hdc.workspace_size(hdc.OP_SEGMENTED_REDUCE, hdc.F32, hdc.ACC_PLAIN, x.numel(), off.numel() - 1),
                     dtype=torch.uint8, device=gpu())
    out = torch.empty(off.numel() - 1, device=gpu())
    eager = hdc.segmented_reduce(x, og, HOR, "plain", ws=ws).clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hdc.segmented_reduce(x, og, HOR, "plain", out=out, ws=ws)
    for _ in range(5):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        hdc.segmented_reduce(x[:1000], og[:20], HOR, "plain", ws=ws)
        torch.cuda.synchronize()
