"""The grouped batch that folds each call's chunk partials in the same launch:
calls of 0, 1, 2, 255, 256 and 257 chunks with ragged ends, more calls than one
group takes, the most chunks that one launch takes and one more, from a
workspace filled with ones, twice in a row (the counters must be back at 0) and
in a replayed graph, against the two-launch form bit for bit and against the
oracle."""
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

CHUNK = 1024
HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}
FAFF, IAFF, IID = {"fn": "affine", "a": 2.5, "b": 0.5}, {"fn": "affine", "a": 3, "b": -7}, {"fn": "identity"}
CLASSES = [(torch.float32, "plain", FAFF, HOR), (torch.bfloat16, "compensated", FAFF, IID),
           (torch.int32, "exact_int", IAFF, IID)]


def value(t):
    return t.cpu().reshape(1).view(torch.int64 if t.element_size() == 8 else torch.int32).item()


@pytest.mark.parametrize("dt,acc,mf,rf", CLASSES, ids=["f32", "bf16", "i32"])
def test_one_launch(dt, acc, mf, rf):
    op, cls = hdc.OP_BATCH, (hdc.DTYPE[dt], hdc.ACC[acc])
    blocks = torch.cuda.get_device_properties(0).multi_processor_count  # grid_mult 1
    lists = [[0, 1, 2, 17], [1] * 33 + [3] * 33, [0, 5, blocks - 7, 0, 2], [5, blocks - 4], [255, 1], [0, 256], [257, 2]]
    saved = [hdc.get_tuning(op, *cls, b) for b in range(hdc.BUCKETS)]
    try:
        for chunks in lists:
            xs = []
            for i, k in enumerate(chunks):
                n = max(0, k * CHUNK - 5 * (i % 2))
                if dt == torch.int32:
                    xs.append(synth.uniform_int(230904800 + i, 0, n, bits=20))
                else:
                    xs.append(synth.to_storage(synth.uniform_pm1_f32(230904800 + i, 0, n).double(), dt))
            xg = [x.cuda() for x in xs]
            total = sum(x.numel() for x in xs)
            ws = torch.empty(hdc.workspace_size(op, *cls, total, len(xs)), dtype=torch.uint8, device="cuda")
            got = {}
            for passes in (2, 1):
                hdc.set_tuning(op, *cls, -1, block=256, unroll=1, grid_mult=1, chunk=CHUNK, passes=passes)
                ws.fill_(0xFF)
                for rep in range(2):
                    got[passes, rep] = [value(v) for v in hdc.batch_map_reduce(xg, mf, rf, acc, ws=ws)[1]]
            assert got[1, 0] == got[1, 1] == got[2, 0] == got[2, 1], chunks
            outs = hdc.batch_map_reduce(xg, mf, rf, acc, ws=ws)[1]
            for v, x in zip(outs, xs):
                ref = oracle.reduce(rf, x)
                if dt == torch.int32:
                    assert v.item() == ref["isum"]
                else:
                    assert abs(v.item() - ref["exact"]) <= 1e-6 * ref["abs_sum"]
            ys, outs = hdc.batch_map_reduce(xg, mf, rf, acc, ws=ws)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                hdc.batch_map_reduce(xg, mf, rf, acc, ys=ys, outs=outs, ws=ws)
            for _ in range(3):
                for v in outs:
                    v.fill_(1)
                graph.replay()
                torch.cuda.synchronize()
                assert [value(v) for v in outs] == got[2, 0], chunks
    finally:
        for b, t in enumerate(saved):
            hdc.set_tuning(op, *cls, b, **t)
