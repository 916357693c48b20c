"""The segmented reduce at the most segments the interface admits (2^31 - 2,
nearly all of them empty): the search over the offsets and the 64 offsets a
wavefront holds at a time must not leave the array, whose last index is the
largest a 32-bit integer holds, less one."""
import pytest
import torch

import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

SEGMENTS = 2 ** 31 - 2


def test_most_segments():
    op, code, acc = hdc.OP_SEGMENTED_REDUCE, hdc.F32, hdc.ACC_PLAIN
    # segment -> its elements: the first, one in the middle, three among the last 64, the last
    filled = {0: 3, SEGMENTS // 2: 1500, SEGMENTS - 61: 2, SEGMENTS - 3: 700, SEGMENTS - 2: 1, SEGMENTS - 1: 5}
    n = sum(filled.values())
    size = hdc.workspace_size(op, code, acc, n, SEGMENTS)
    if torch.cuda.mem_get_info()[0] < size + 12 * SEGMENTS + (8 << 30):
        pytest.skip("needs 140 GB of free device memory")
    x = torch.arange(1, n + 1, dtype=torch.float32, device="cuda")
    off = torch.zeros(SEGMENTS + 1, dtype=torch.int64, device="cuda")
    want, at = {}, 0
    for j, length in filled.items():
        off[j + 1:] += length
        want[j] = float(sum(range(at + 1, at + length + 1)))  # an integer below 2^24: exact in any order
        at += length
    out = torch.full((SEGMENTS,), 77.0, device="cuda")
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    print(f"most segments: S={SEGMENTS} n={n} workspace={size}", flush=True)
    hdc.segmented_reduce(x, off, {"fn": "identity"}, "plain", out=out, ws=ws)
    got = {j: out[j].item() for j in filled}
    nonzero = sum(torch.count_nonzero(part).item() for part in out.split(1 << 28))
    del off, out, ws
    torch.cuda.empty_cache()
    assert got == want
    assert nonzero == len(filled)
