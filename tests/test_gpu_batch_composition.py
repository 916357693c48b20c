"""The reduction of a batch's call has the same bits whatever other calls the
batch holds: alone, among small calls, and beside one so large that the average
call changes its size bucket; for calls of every bucket, under the shipped
tuning cache."""
import pytest
import torch

import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

HOR, IDENT = {"fn": "horner", "coef": synth.horner_coefficients(8)}, {"fn": "identity"}
AFF = {"fn": "affine", "a": 2.5, "b": 0.5}
CLASSES = [(torch.float32, "plain", HOR), (torch.float32, "compensated", IDENT), (torch.float16, "plain", HOR),
           (torch.float16, "compensated", HOR), (torch.bfloat16, "plain", IDENT), (torch.bfloat16, "compensated", IDENT)]
SIZES = [50_001, 300_007, 2_000_003, 17_000_001]  # one per size bucket


@pytest.mark.parametrize("dt,acc,fn", CLASSES, ids=[f"{str(c[0])[6:]}_{c[1]}" for c in CLASSES])
def test_bits_do_not_depend_on_the_other_calls(dt, acc, fn):
    g = torch.Generator(device="cuda").manual_seed(230905400)
    xs = [torch.empty(n, device="cuda").uniform_(-1, 1, generator=g).to(dt) for n in SIZES]
    small = [torch.ones(100 + i, dtype=dt, device="cuda") for i in range(20)]
    huge = torch.ones(1 << 27, dtype=dt, device="cuda")

    def fold(batch, at):
        return hdc.batch_map_reduce(batch, None, fn, acc)[1][at].item()

    for x in xs:
        print(f"batch composition {dt} {acc} n={x.numel()}", flush=True)
        got = [fold([x], 0), fold(small + [x], 20), fold([huge, x], 1), fold(xs + [x], 4), fold(xs + [huge, x], 5),
               hdc.batch_map_reduce([huge, x], AFF, fn, acc)[1][1].item()]
        assert len(set(got)) == 1, (x.numel(), got)
