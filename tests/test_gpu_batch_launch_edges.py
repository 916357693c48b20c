"""The edges at which a grouped batch stops folding in the same launch: 64
chunks in one call, as many chunks in all as compute units, counted in the
chunks that each storage type really gets (whole block steps).  One launch
against two bit for bit and against the oracle; which form runs is read off the
nodes of the captured call."""
import ctypes

import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

BLOCK = 256
HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}
FAFF, IAFF, IID = {"fn": "affine", "a": 2.5, "b": 0.5}, {"fn": "affine", "a": 3, "b": -7}, {"fn": "identity"}
CLASSES = [(torch.float32, "plain", FAFF, HOR), (torch.float16, "compensated", FAFF, HOR),
           (torch.bfloat16, "compensated", FAFF, IID), (torch.int32, "exact_int", IAFF, IID)]


def lists(cus):
    """(chunks per call, one launch)"""
    full = [64] * ((cus - 1) // 64)
    rest = cus - sum(full)
    return [([64], True), ([65], False), ([64, 63, 1], True), ([64, 65, 1], False), (full + [rest], True),
            (full + [rest, 1], False), ([1, 0, rest - 1] + full, True), ([2, 0, rest - 1] + full, False),
            ([1] * 31 + [64, 2, 0], True)]  # the 33rd call is a group of its own


def value(t):
    return t.cpu().reshape(1).view(torch.int64 if t.element_size() == 8 else torch.int32).item()


def launches(call):
    """Kernel launches of a call: the nodes of its capture."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64.so" in line))
    nodes = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
    return nodes.value


@pytest.mark.parametrize("dt,acc,mf,rf", CLASSES, ids=["f32", "f16", "bf16", "i32"])
def test_edges(dt, acc, mf, rf):
    op, cls = hdc.OP_BATCH, (hdc.DTYPE[dt], hdc.ACC[acc])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    vec = 4 if dt in (torch.float32, torch.int32) else 8
    chunk = max(1024, BLOCK * vec)  # a chunk of 1024 elements, in whole steps of BLOCK vectors
    saved = [hdc.get_tuning(op, *cls, b) for b in range(hdc.BUCKETS)]
    try:
        for chunks, one in lists(cus):
            sizes = [max(0, k * chunk - 5 * (i % 2)) for i, k in enumerate(chunks)]
            if dt == torch.int32:
                xs = [synth.uniform_int(230905500 + i, 0, n, bits=20) for i, n in enumerate(sizes)]
            else:
                xs = [synth.to_storage(synth.uniform_pm1_f32(230905500 + i, 0, n).double(), dt)
                      for i, n in enumerate(sizes)]
            xg = [x.cuda() for x in xs]
            ws = torch.empty(hdc.workspace_size(op, *cls, sum(sizes), len(xs)), dtype=torch.uint8, device="cuda")
            got = {}
            for passes in (2, 1):
                hdc.set_tuning(op, *cls, -1, block=BLOCK, unroll=1, grid_mult=2, chunk=1024, passes=passes)
                ws.fill_(0xFF)
                print(f"batch edges {dt} {chunks} passes={passes}", flush=True)
                for rep in range(2):
                    got[passes, rep] = [value(v) for v in hdc.batch_map_reduce(xg, mf, rf, acc, ws=ws)[1]]
            assert got[1, 0] == got[1, 1] == got[2, 0] == got[2, 1], chunks
            ys, outs = hdc.batch_map_reduce(xg, mf, rf, acc, ws=ws)
            groups = (len(xs) + 31) // 32
            count = launches(lambda: hdc.batch_map_reduce(xg, mf, rf, acc, ys=ys, outs=outs, ws=ws))
            assert count == groups if one else count > groups, (chunks, count)
            for v, y, x in zip(outs, ys, xs):
                ref = oracle.reduce(rf, x)
                if dt == torch.int32:
                    assert v.item() == ref["isum"]
                else:
                    assert abs(v.item() - ref["exact"]) <= 1e-6 * ref["abs_sum"]
                iv = torch.int32 if dt.itemsize == 4 else torch.int16
                assert torch.equal(y.cpu().view(iv), oracle.map(mf, x).view(iv))
    finally:
        for b, t in enumerate(saved):
            hdc.set_tuning(op, *cls, b, **t)
