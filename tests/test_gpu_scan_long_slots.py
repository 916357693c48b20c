"""Single-pass scans of more than 256 tiles, whose look-back nodes lie in the
library's long slots up to 16384 tiles and in the workspace beyond: three tree
levels, the last tile count of a slot and the first past it, rising and falling
sizes on one workspace filled with ones, plain and segmented, and more
workspaces than there are slots.  The inputs are small integers, so every fold
order gives the exact prefix sums and the comparison is bit for bit."""
import numpy as np
import pytest
import torch

import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

TILE = 64 * 16
COUNTS = [16385, 257, 16384, 4097, 256, 16384]
IDENT = {"fn": "identity"}
CLASSES = [(torch.int32, "exact_int"), (torch.float32, "plain"), (torch.bfloat16, "compensated")]


@pytest.fixture(autouse=True)
def small_tiles():
    keys = [(hdc.DTYPE[dt], hdc.ACC[acc], b) for dt, acc in CLASSES for b in range(hdc.BUCKETS)]
    saved = {k: hdc.get_tuning(hdc.OP_SCAN, *k) for k in keys}
    for dt, acc in CLASSES:
        hdc.set_tuning(hdc.OP_SCAN, hdc.DTYPE[dt], hdc.ACC[acc], -1, block=64, unroll=4)
    yield
    for k, t in saved.items():
        hdc.set_tuning(hdc.OP_SCAN, *k, **t)


def workspace(n):
    size = hdc.workspace_size(hdc.OP_SCAN, hdc.I32, hdc.ACC_EXACT_INT, n)
    return torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("dt,acc", CLASSES, ids=["i32", "f32", "bf16"])
def test_tile_counts(dt, acc):
    ints = torch.randint(-100, 101, (max(COUNTS) * TILE,), generator=torch.Generator().manual_seed(230904900))
    sums = torch.cat([torch.zeros(1, dtype=torch.int64), ints.cumsum(0)])
    x = ints.to(dt).cuda()
    ws = workspace(ints.numel())
    for tiles in COUNTS:
        n = tiles * TILE - 7
        off = torch.tensor([0, n // 3, n // 3, n - 5 * TILE, n], dtype=torch.int64)
        start = torch.repeat_interleave(sums[off[:-1]], off.diff())
        print(f"scan long slots {dt} tiles={tiles}", flush=True)
        y = hdc.scan(x[:n], IDENT, acc, True, ws=ws)
        assert np.array_equal(y.cpu().numpy(), sums[:n].to(y.dtype).numpy()), tiles
        z = hdc.segmented_scan(x[:n], off.cuda(), IDENT, acc, False, ws=ws)
        assert np.array_equal(z.cpu().numpy(), (sums[1:n + 1] - start).to(z.dtype).numpy()), tiles


def test_more_workspaces_than_slots():
    n = 300 * TILE + 1
    x = torch.randint(-100, 101, (n,), generator=torch.Generator().manual_seed(230904901), dtype=torch.int32).cuda()
    want = torch.cumsum(x.long(), 0)
    spaces = [workspace(n) for _ in range(40)]
    for rep in range(2):
        for ws in spaces:
            assert torch.equal(hdc.scan(x, IDENT, "exact_int", ws=ws), want), rep
