"""The one-launch fold at the edges of its ticket: one block (no ticket), up to
two arrival groups counted on the root alone, the fan of 16 counters from 33
blocks on, full and ragged groups, and a grid at the tuning's cap.  Every fold
state, from a workspace filled with ones (nothing in it may be relied on), two
calls in a row (the ticket must be back at 0), against the two-launch form bit
for bit and against the oracle."""
import pytest
import torch

import oracle
import paper_2309_03912_amd as hdc
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-6
HORNER = {"fn": "horner", "coef": synth.horner_coefficients(8)}
IDENT, PROD = {"fn": "identity"}, {"fn": "product"}
CASES = [
    ("f32_plain", hdc.OP_TRANSFORM_REDUCE, torch.float32, HORNER, "plain"),
    ("bf16_comp", hdc.OP_TRANSFORM_REDUCE, torch.bfloat16, IDENT, "compensated"),
    ("i32", hdc.OP_TRANSFORM_REDUCE, torch.int32, IDENT, "exact_int"),
    ("f16_exact", hdc.OP_TRANSFORM_REDUCE, torch.float16, IDENT, "exact"),
    ("bf16_exact", hdc.OP_TRANSFORM_REDUCE, torch.bfloat16, IDENT, "exact"),
    ("f16_dot_exact", hdc.OP_DOT, torch.float16, PROD, "exact"),
]


@pytest.mark.parametrize("name,op,dt,fn,acc", CASES, ids=[c[0] for c in CASES])
def test_ticket_edges(name, op, dt, fn, acc):
    dev = torch.device("cuda", 0)
    code, a = hdc.DTYPE[dt], hdc.ACC[acc]
    per_block = 64 * (4 if dt in (torch.float32, torch.int32) else 8)  # block 64, one 16-byte vector per lane
    saved = {b: hdc.get_tuning(op, code, a, b) for b in range(hdc.BUCKETS)}
    blocks = [1, 2, 16, 17, 32, 33, 34, 48, 49, 255, 512, 2049]
    n_max = blocks[-1] * per_block
    if dt == torch.int32:
        x = synth.uniform_int(230903990, 0, n_max, bits=20)
    else:
        x = synth.to_storage(synth.normal_f64(230903990, 0, n_max), dt)
    z = synth.to_storage(synth.normal_f64(230903990, 1, n_max), dt) if fn is PROD else None
    xg, zg = x.to(dev), z.to(dev) if z is not None else None
    ws = torch.empty(hdc.workspace_size(hdc.OP_TRANSFORM_REDUCE, code, a, n_max), dtype=torch.uint8, device=dev)
    try:
        for g in blocks:
            n = g * per_block - 3  # g blocks, a ragged last vector
            zn = zg[:n] if zg is not None else None
            got = {}
            for passes in (2, 1):
                hdc.set_tuning(op, code, a, -1, block=64, unroll=1, grid_mult=64, passes=passes)
                ws.fill_(0xFF)
                print(f"ticket edges {name} blocks={g} passes={passes}", flush=True)
                got[passes] = [hdc.transform_reduce(xg[:n], fn, acc, z=zn, ws=ws) for _ in range(2)]
            torch.cuda.synchronize()
            vals = [v.cpu().reshape(1).view(torch.int64 if v.element_size() == 8 else torch.int32).item()
                    for v in got[2] + got[1]]
            assert len(set(vals)) == 1, (name, g, vals)
            ref = oracle.reduce(fn, x[:n], z[:n] if z is not None else None)
            v = got[1][0].item()
            if acc == "exact_int":
                assert v == ref["isum"], (name, g)
            elif acc == "exact":
                assert v == ref["exact"], (name, g)
            else:
                assert abs(v - ref["exact"]) <= TOL * ref["abs_sum"], (name, g)
    finally:
        for b, t in saved.items():
            hdc.set_tuning(op, code, a, b, **t)


@pytest.mark.parametrize("dt", [torch.float16, torch.bfloat16])
def test_exact_rounding_edges(dt):
    """Exact sums whose rounding to fp64 is a tie, just off a tie, or carries into the next binade, and
    sums of one bit: the result equals the oracle's correctly rounded sum."""
    dev = torch.device("cuda", 0)
    big = 32768.0 if dt == torch.float16 else 2.0 ** 60
    tiny = 2.0 ** -24 if dt == torch.float16 else 2.0 ** -133
    cases = [[tiny], [-tiny], [big, tiny], [big, -tiny], [big] * 4096 + [tiny], [-big] * 4096 + [-tiny] * 3]
    if dt == torch.bfloat16:
        for top in (2.0 ** 60, -2.0 ** 100, 2.0 ** -40):  # 53 bits end at top * 2^-52: half of it is the tie
            h = abs(top) * 2.0 ** -53
            for low in ([h], [h, h * 2.0 ** -20], [h, -h * 2.0 ** -20], [h] * 3, [h] * 3 + [-h * 2.0 ** -30]):
                cases.append([top] + low)
    else:  # 2^14 terms of 32768 reach 2^29; units of 2^-24 give at most 53 bits, so 2^20 terms are needed for a tie
        cases += [[big] * (1 << 15) + [tiny] * k for k in (1, 2, 3)]
    for c in cases:
        x = torch.tensor(c, dtype=torch.float64).to(torch.float32).to(dt)
        got = hdc.transform_reduce(x.to(dev), IDENT, "exact").item()
        ref = oracle.reduce(IDENT, x)["exact"]
        assert got == ref, (dt, c[:4], len(c), got, ref)
