"""GPU: BC7 blocks so near a line that bounds rule nothing out, which go without
them sixteen at a time: bit-exact against the oracle's exhaustive search where
sixteens are whole, broken by one other block, or ragged, and where every block
of a window stays in the search."""
import numpy as np
import pytest

import oracle as O
from test_gpu_bc7_search import _blocks, _prim_desc


def _flat(n, seed, every):
    """Two adjacent levels a channel; every `every`-th block of other kinds."""
    t = _blocks("near_constant", n, seed)
    for k, kind in enumerate(("random", "gradient", "constant", "two_level")):
        at = np.arange(3 + k * every, n, 4 * every)
        t[at] = _blocks(kind, n, seed + 1 + k)[at]
    return t


@pytest.mark.gpu
@pytest.mark.parametrize("nblk,every", [(528, 10_000), (528, 17), (272, 16), (112, 40)])
def test_flat_blocks_equal_exhaustive(nblk, every):
    import torch
    from paper_2607_14513_amd import gsbc
    t = _flat(nblk, 31, every)
    want, sse = O.bc7_encode(t)
    with gsbc.Context(0) as ctx:
        out, _, s = ctx.encode(torch.from_numpy(t[None]).cuda(), _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7, want_sse=True)
    assert np.array_equal(out.cpu().numpy()[:16 * nblk].reshape(-1, 16), want.reshape(-1, 16))
    assert s[1][0] == int(np.asarray(sse, np.int64).sum())


@pytest.mark.gpu
@pytest.mark.parametrize("mask", [0xFF, 0x02, 0x05])
def test_whole_windows_stay(mask):
    import torch
    from paper_2607_14513_amd import gsbc
    unit, nblk = 512, (1 << 17) + 272
    t = _flat(unit, 32, 10_000)
    want, _ = O.bc7_encode(t, mode_mask=mask)
    with gsbc.Context(0) as ctx:
        tex = torch.from_numpy(t).cuda().repeat(-(-nblk // unit), 1, 1)[:nblk].contiguous()
        out, _, _ = ctx.encode(tex[None], _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7, params=gsbc.default_params(bc7_mode_mask=mask))
    got = out.cpu().numpy()[:16 * nblk].reshape(-1, 16)
    assert np.array_equal(got, np.tile(want.reshape(-1, 16), (-(-nblk // unit), 1))[:nblk])
