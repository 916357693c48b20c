"""A segmented reduce without a workspace argument gives the same bits whatever
the calls before it were: the binding's cached buffer grows with them, but a
call plans for its own elements only."""
import numpy as np
import pytest
import torch

import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

HOR = {"fn": "horner", "coef": synth.horner_coefficients(8)}


@pytest.mark.parametrize("mean", [20, 3000])
def test_same_bits_after_a_larger_call(mean):
    rng = np.random.default_rng(230905800)
    off = synth.offsets_from_lengths(torch.as_tensor(rng.integers(0, 2 * mean, 600_000 // mean), dtype=torch.int64))
    x = torch.as_tensor(rng.standard_normal(int(off[-1])), dtype=torch.float32).cuda()
    large = torch.ones(60_000_000, device="cuda")
    few = torch.tensor([0, 5, 60_000_000], device="cuda")
    off = off.cuda()
    stream = torch.cuda.Stream()  # a stream of its own has a buffer of its own
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        first = hdc.segmented_reduce(x, off, HOR, "plain").clone()
        hdc.segmented_reduce(large, few, HOR, "plain")
        hdc.transform_reduce(x, HOR, "plain")
        second = hdc.segmented_reduce(x, off, HOR, "plain").clone()
        torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int32), second.view(torch.int32))
