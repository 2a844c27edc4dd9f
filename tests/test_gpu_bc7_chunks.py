"""GPU: where the BC7 encoder's scratch for a whole chunk cannot be had, smaller
chunks are taken, with the same bits; only when the smallest cannot does the
call report GSBC_E_NOMEM.  In fresh processes (the injected failures count per
process)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CODE = """
import ctypes, os, sys
import torch
from paper_2607_14513_amd import gsbc
n = 150_064
t = torch.randint(0, 256, (1, n, 16, 4), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
d = gsbc.StreamDesc()
d.n_prims = d.n_pad = d.blocks_per_stream = n
d.arrangement, d.n_streams, d.format[0] = gsbc.ARR_PRIM, 1, gsbc.FMT_BC7
for k in range(16):
    d.vmin[k], d.vmax[k] = 0.0, 1.0
st = torch.cuda.Stream()
torch.cuda.synchronize()
def one(batch):
    with gsbc.Context(0, stream=st) as ctx, torch.cuda.stream(st):
        if batch:
            out = torch.empty(16 * n, dtype=torch.uint8, device="cuda")
            ctx.encode_batch([t], [d], [out])
        else:
            out = ctx.encode(t, d, fmt=gsbc.FMT_BC7)[0][:16 * n]
        ctx.sync()
        return out.clone(), ctx.arena_info()[0]
batch = sys.argv[1] == "batch"
got, small = one(batch)                  # its first allocation fails
ref, large = one(batch)
torch.cuda.synchronize()
assert torch.equal(got, ref)
assert batch or small < large, (small, large)
print("SAME")
"""


@pytest.mark.parametrize("call", ["encode", "batch"])
def test_smaller_chunks(call):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, GSBC_FAULT="alloc:1", PYTHONPATH=root)
    r = subprocess.run([sys.executable, "-c", CODE, call], env=env, cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "SAME" in r.stdout, r.stderr[-2000:]


@pytest.mark.parametrize("n", [100, 5_000, 3_000_000])
def test_reserve_allocates_once(n):
    from paper_2607_14513_amd import gsbc
    with gsbc.Context(0) as ctx:
        ctx.reserve(n)
        size, growths = ctx.arena_info()
        assert growths == 1
        ctx.reserve(n)
        assert ctx.arena_info() == (size, 1)
