"""A few elements in many segments, most of them empty, with a workspace sized
for far more: the one tile is crowded, and of fewer elements than the parts it
is cut into, so that some parts hold nothing; every storage type and fold,
whole numbers whose sums are exact."""
import numpy as np
import pytest
import torch

import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

CLASSES = [(torch.float32, "plain"), (torch.float32, "compensated"), (torch.bfloat16, "plain"),
           (torch.bfloat16, "compensated"), (torch.float16, "compensated"), (torch.int32, "exact_int")]


def layouts():
    rng = np.random.default_rng(230905310)
    for n in (1, 2, 3, 7, 8, 9, 63, 64, 127, 128, 129, 500):
        for S in (65, 250, 2000):
            yield f"{n}_in_{S}", np.diff(np.concatenate([[0], np.sort(rng.integers(0, n + 1, S - 1)), [n]]))
        yield f"{n}_at_the_end", [0] * 300 + [n]
        yield f"{n}_at_the_start", [n] + [0] * 300
        yield f"{n}_ones", [0] * 70 + [1] * n + [0] * 70


@pytest.mark.parametrize("dt,acc", CLASSES, ids=[f"{str(c[0])[6:]}_{c[1]}" for c in CLASSES])
@pytest.mark.parametrize("chunk", [None, 65536])
def test_few_elements(dt, acc, chunk):
    op, code, a = hdc.OP_SEGMENTED_REDUCE, hdc.DTYPE[dt], hdc.ACC[acc]
    saved = {b: hdc.get_tuning(op, code, a, b) for b in range(hdc.BUCKETS)}
    if chunk:
        hdc.set_tuning(op, code, a, -1, chunk=chunk)
    try:
        for name, L in layouts():
            for start, shift in ((0, 0), (2, 8), (3, 1)):
                print(f"few {name} {dt} {acc} chunk={chunk} start={start} shift={shift}", flush=True)
                off = np.concatenate([[0], np.cumsum(L)]) + start
                v = np.arange(off[-1] + 3) % 17 - 8
                want = [int(v[s:e].sum()) for s, e in zip(off[:-1], off[1:])]
                x = torch.as_tensor(np.concatenate([np.zeros(shift, dtype=v.dtype), v])).to(dt).cuda()[shift:]
                ws = torch.full((hdc.workspace_size(op, code, a, 500_000_000, len(want)),), 0xFF, dtype=torch.uint8,
                                device="cuda")
                out = torch.full((len(want),), 77, dtype=hdc.OUT_DTYPE[a], device="cuda")
                hdc.segmented_reduce(x, torch.as_tensor(off, device="cuda"), {"fn": "identity"}, acc, out=out, ws=ws)
                assert out.cpu().tolist() == want, name
    finally:
        for b, t in saved.items():
            hdc.set_tuning(op, code, a, b, **t)
