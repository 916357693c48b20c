"""A process that has used up the library's tickets (one per workspace and
stream): one-launch reductions, batches and segmented reduces with a new
workspace fold in a second launch, and give the same bits as before.  In a
child process, so that the tests of this one keep their tickets."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = r"""
import sys
import numpy as np
import torch
import paper_2309_03912_amd as hdc
import synth

COEF = synth.horner_coefficients(8)
HOR, IDENT, PROD = {"fn": "horner", "coef": COEF}, {"fn": "identity"}, {"fn": "product"}
AFF = {"fn": "affine", "a": 2.5, "b": 0.5}
rng = np.random.default_rng(230905200)
x32 = torch.as_tensor(rng.standard_normal(900_001), dtype=torch.float32).cuda()
x16, xb = x32.to(torch.float16), x32.to(torch.bfloat16)
off = synth.offsets_from_lengths(torch.as_tensor(rng.integers(0, 9000, 200), dtype=torch.int64)).clamp(max=900_000)
off[-1] = 900_000
rows = synth.offsets_from_lengths(torch.as_tensor(rng.integers(0, 50, 30_000), dtype=torch.int64)).clamp(max=900_000)
off, rows = off.cuda(), rows.cuda()
calls = {
    "sum f32": lambda ws: [hdc.transform_reduce(x32, HOR, "plain", ws=ws)],
    "sum bf16 exact": lambda ws: [hdc.transform_reduce(xb, IDENT, "exact", ws=ws)],
    "dot f16": lambda ws: [hdc.transform_reduce(x16, PROD, "compensated", z=x16, ws=ws)],
    "dot f16 exact": lambda ws: [hdc.transform_reduce(x16, PROD, "exact", z=x16, ws=ws)],
    "map_reduce": lambda ws: list(hdc.map_reduce(x16, AFF, HOR, "compensated", ws=ws)),
    "batch": lambda ws: hdc.batch_map_reduce([x32[:70_000], x32[:5]], AFF, HOR, "plain", ws=ws)[1],
    "segmented f32": lambda ws: [hdc.segmented_reduce(x32, off, IDENT, "plain", ws=ws)],
    "segmented f32 rows": lambda ws: [hdc.segmented_reduce(x32, rows, HOR, "plain", ws=ws)],
    "segmented bf16": lambda ws: [hdc.segmented_reduce(xb, off, IDENT, "compensated", ws=ws)],
    "scan f32": lambda ws: [hdc.scan(x32[:100_000], IDENT, "plain", ws=ws)],
}
size = max(hdc.workspace_size(op, hdc.F32, 0, 900_001, 30_000) for op in range(7)) // 256 * 256 + 256
segsize = {k: hdc.workspace_size(hdc.OP_SEGMENTED_REDUCE, hdc.F32, 0, 900_001, s)
           for k, s in (("segmented f32", 200), ("segmented bf16", 200), ("segmented f32 rows", 30_000))}
spaces = [torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda") for _ in range(2)]
got = [{}, {}]
for k, ws in enumerate(spaces):
    if k == 1:  # use up the tickets: 70,000 workspaces 256 bytes apart
        need = hdc.workspace_size(hdc.OP_TRANSFORM_REDUCE, hdc.F32, 0, 1000)
        buf = torch.empty(need + 70_000 * 256, dtype=torch.uint8, device="cuda")
        out = torch.empty((), device="cuda")
        for i in range(70_000):
            hdc.transform_reduce(x32[:1000], IDENT, "plain", out=out, ws=buf[256 * i:256 * i + need])
        torch.cuda.synchronize()
    for name, call in calls.items():
        print("no ticket left:", k, name, flush=True)
        got[k][name] = [t.cpu() for t in call(ws[:segsize[name]] if name in segsize else ws)]
for name in calls:
    for a, b in zip(got[0][name], got[1][name]):
        assert np.array_equal(a.reshape(-1).view(torch.uint8).numpy(), b.reshape(-1).view(torch.uint8).numpy()), name
print("SAME_BITS", flush=True)
"""


def test_same_bits_without_a_ticket():
    run = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=ROOT, env=dict(os.environ, PYTHONPATH=ROOT),
                         capture_output=True, text=True, timeout=100)
    print(run.stdout[-2000:], run.stderr[-2000:])
    assert run.returncode == 0 and "SAME_BITS" in run.stdout


MANY = r"""
import torch
import paper_2309_03912_amd as hdc

x = torch.rand(100_000, device="cuda")
out = torch.empty((), device="cuda")
need = hdc.workspace_size(hdc.OP_TRANSFORM_REDUCE, hdc.F32, 0, 100_000)
buf = torch.empty(need + 60_000 * 256, dtype=torch.uint8, device="cuda")
want = hdc.transform_reduce(x, {"fn": "identity"}, "plain").item()
got = torch.empty(60_000, device="cuda")
for rep in range(2):  # twice: every ticket is back at 0
    got.fill_(float("nan"))
    for i in range(60_000):
        hdc.transform_reduce(x, {"fn": "identity"}, "plain", out=got[i], ws=buf[256 * i:256 * i + need])
    assert (got == want).all().item(), rep
print("SAME_SUMS", flush=True)
"""


def test_sixty_thousand_workspaces_take_one_launch():
    """A program whose workspaces change address (a caching allocator) keeps the one-launch form."""
    run = subprocess.run([sys.executable, "-u", "-c", MANY], cwd=ROOT,
                         env=dict(os.environ, PYTHONPATH=ROOT, HDC_LOG="1"), capture_output=True, text=True, timeout=100)
    lines = [v for v in run.stderr.splitlines() if v.startswith("hdc: transform_reduce")]
    print(run.stdout[-500:], run.stderr[-500:])
    assert run.returncode == 0 and "SAME_SUMS" in run.stdout
    assert len(lines) == 120_001 and all("schedule=one launch" in v for v in lines)
