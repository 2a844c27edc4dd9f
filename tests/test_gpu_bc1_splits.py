"""The BC1 cluster fit scores only the splits whose lower bound leaves them a
chance, 64 of a wave's queued splits at a time: bit-exact against the oracle's
exhaustive fit on waves that mix constant and other blocks, that queue few
splits or nearly all (scored in uniform order then), with ties between splits
and ragged waves, with the four waves of a small encode sharing their blocks and
for every workgroup size."""
import numpy as np
import pytest

import oracle as O
from conftest import rgba, smooth_blocks
from test_gpu_bc7_search import _blocks, _prim_desc


def _mixed(n, seed):
    """Constant, two-coloured, smooth, gradient and random blocks in turn."""
    kinds = ["near_constant", "two_level", "gradient", "one_channel", "corners", "random"]
    t = np.concatenate([_blocks(k, n, seed)[None] for k in kinds] + [smooth_blocks(n, seed, 2)[None]])
    out = np.moveaxis(t, 0, 1).reshape(-1, 16, 4)[:n].copy()
    out[::5] = out[::5, :1]
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("lanes", [0, 64, 128, 256])   # 0: shared blocks (one round per item)
@pytest.mark.parametrize("kind,nblk", [("mixed", 1040), ("gradient", 272), ("near_constant", 272), ("two_level", 272),
                                       ("one_channel", 272), ("corners", 272), ("smooth", 272), ("random", 16),
                                       ("constant", 80)])
def test_splits_equal_exhaustive(kind, nblk, lanes):
    import torch
    from paper_2607_14513_amd import gsbc
    t = _mixed(nblk, 21) if kind == "mixed" else smooth_blocks(nblk, 22, 12) if kind == "smooth" else \
        rgba(np.repeat(np.random.default_rng(23).integers(0, 256, (nblk, 1, 3)), 16, 1)) if kind == "constant" else \
        _blocks(kind, nblk, 24)
    want, _ = O.bc1_encode(t)
    d = _prim_desc(gsbc, nblk)
    d.format[0] = gsbc.FMT_BC1
    s = torch.cuda.Stream()
    with gsbc.Context(0, stream=s) as ctx:
        tex = torch.from_numpy(t[None]).cuda()
        out = torch.empty(8 * nblk, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        ctx.encode_batch([tex], [d], [out], tuning=gsbc.default_batch_tuning(bc1_lanes=lanes or 128, item_rounds=2 if lanes else 1))
        ctx.sync()
        assert np.array_equal(out.cpu().numpy().reshape(-1, 8), np.asarray(want).reshape(-1, 8))
