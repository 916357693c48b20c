"""Rounding of the scans that take 32 elements per thread (plain folds of 2^25
elements and more): uniform and one-signed values, f32 and 16-bit storage,
every prefix against the fp64 prefix sum within the library's tolerance (1e-6
of the sum of magnitudes so far).  A tile's 32,768 elements are folded in fp32
as a lane's run of 4 or 8, a scan over 64 lanes, and chains over at most 8
chunks and 16 wavefronts: 8 + 6 + 8 + 16 roundings of 2^-24 of that sum at most,
2.3e-6, and in practice (their signs vary) far less; the carry is fp64."""
import pytest
import torch

import paper_2309_03912_amd as hdc

pytestmark = pytest.mark.gpu

N = (1 << 25) + 12_345
TOL = 1e-6


@pytest.mark.parametrize("low", [-1.0, 0.0], ids=["both_signs", "one_sign"])
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
def test_rounding(dt, low):
    g = torch.Generator(device="cuda").manual_seed(230905700)
    x = torch.empty(N, device="cuda").uniform_(low, 1.0, generator=g).to(dt)
    want = torch.cumsum(x.double(), 0)
    bound = TOL * torch.cumsum(x.double().abs(), 0)
    for exclusive in (False, True):
        y = hdc.scan(x, {"fn": "identity"}, "plain", exclusive).double()
        ref, tol = (want - x.double(), bound) if exclusive else (want, bound)
        err = (y - ref).abs()
        # the output itself is fp32: half a unit in the last place of the prefix
        assert torch.all(err <= tol + ref.abs() * 2.0 ** -24), (exclusive, (err / bound).max().item())
        print(f"wide rounding {dt} low={low} exclusive={exclusive}: "
              f"{(err / bound).max().item():.3f} of the tolerance", flush=True)
