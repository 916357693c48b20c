"""Single-pass scans around 2^25 elements, where plain and int64 folds change
from 16 to 32 elements per thread: one element below, the limit, and ragged
ends of 1 and half a tile above it, inclusive and exclusive, 2-byte storage on
and off 4-byte boundaries, the smallest and the largest tile.  The inputs are
small integers, so every fold order gives the exact prefix sums and the
comparison is bit for bit."""
import numpy as np
import pytest
import torch

import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

LIMIT = 1 << 25
IDENT = {"fn": "identity"}
CLASSES = [(torch.int32, "exact_int"), (torch.float32, "plain"), (torch.bfloat16, "plain"), (torch.float16, "plain")]


@pytest.mark.parametrize("block", [64, 1024])
@pytest.mark.parametrize("dt,acc", CLASSES, ids=["i32", "f32", "bf16", "f16"])
def test_around_the_limit(dt, acc, block):
    op, cls = hdc.OP_SCAN, (hdc.DTYPE[dt], hdc.ACC[acc])
    saved = [hdc.get_tuning(op, *cls, b) for b in range(hdc.BUCKETS)]
    ints = torch.randint(-100, 101, (LIMIT + block * 16 + 9,), generator=torch.Generator().manual_seed(230904700))
    sums = torch.cat([torch.zeros(1, dtype=torch.int64), ints.cumsum(0)])
    try:
        hdc.set_tuning(op, *cls, -1, block=block, unroll=4)
        for n, shift, exclusive in [(LIMIT - 1, 0, False), (LIMIT, 0, True), (LIMIT + 1, 0, False), (LIMIT + 1, 1, True),
                                    (LIMIT + block * 16 + 7, 0, True), (LIMIT + block * 16 + 7, 2, False)]:
            x = ints.to(dt).cuda()[shift:shift + n]
            y = hdc.scan(x, IDENT, acc, exclusive=exclusive)
            ref = sums[shift:shift + n] if exclusive else sums[shift + 1:shift + n + 1]
            ref = (ref - sums[shift]).to(y.dtype)
            assert np.array_equal(y.cpu().numpy(), ref.numpy()), (n, shift, exclusive)
    finally:
        for b, t in enumerate(saved):
            hdc.set_tuning(op, *cls, b, **t)
