"""The in-place update's column slices: the head counts at which their number
changes, chunks of rows that end inside a slice's chunk or fill it exactly,
and strided heads, against the oracle's gather of the cache (rows are copies:
bit for bit, nothing else written)."""

import numpy as np
import pytest
import torch

from oracle import compact as o_compact
from paper_2408_03675_amd import nacl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,L,C,D,dt,blhd", [
    (1, 300, 1, 64, "bf16", False),
    (1, 20011, 8193, 128, "bf16", False),
    (3, 9000, 4096, 128, "f32", False),
    (5, 9000, 4097, 64, "f32", True),
    (8, 2100, 1025, 128, "bf16", True),
    (16, 2100, 2099, 64, "bf16", False),
    (31, 700, 257, 128, "f32", False),
    (32, 3000, 1024, 128, "bf16", False),
    (64, 700, 511, 128, "bf16", True),
    (127, 600, 129, 64, "bf16", False),
    (128, 600, 512, 128, "bf16", False),
    (257, 300, 131, 128, "bf16", False),
    # whole rows: chunks of 1024, 512 and 256 rows (8, 16 and 32 vectors a row) and one more
    (130, 1100, 1025, 64, "bf16", False),
    (65, 600, 513, 128, "bf16", True),
    (40, 400, 257, 128, "f32", False),
    (300, 300, 256, 128, "f32", False),
])
def test_in_place_slices(heads, L, C, D, dt, blhd):
    print("in place", heads, L, C, D, dt, blhd, flush=True)
    rng = np.random.default_rng(heads * 1000 + L)
    tdt, view = (torch.bfloat16, torch.int16) if dt == "bf16" else (torch.float32, torch.int32)
    shape = (1, L, heads, D) if blhd else (1, heads, L, D)
    k, v = (torch.randn(shape, device="cuda").to(tdt) for _ in range(2))
    if blhd:
        k, v = k.permute(0, 2, 1, 3), v.permute(0, 2, 1, 3)
    idx = np.stack([np.sort(rng.choice(L, C, replace=False)) for _ in range(heads)])[None]
    idx[0, 0] = np.arange(C)                 # nothing moves
    if heads > 2:
        idx[0, 1] = np.arange(L - C, L)      # every row moves
    kb, vb = (t.contiguous().cpu().view(view).numpy() for t in (k, v))
    prob = nacl.Problem.from_tensors(k, k, v, [L - 1])
    nacl.compact(prob, k, v, torch.from_numpy(idx.astype(np.int32)).cuda(), in_place=True)
    torch.cuda.synchronize()
    kr, vr = o_compact(kb, vb, idx)
    for got, ref, before in ((k, kr, kb), (v, vr, vb)):
        got = got.contiguous().cpu().view(view).numpy()
        assert np.array_equal(got[:, :, :C], ref)
        assert np.array_equal(got[:, :, C:], before[:, :, C:])
