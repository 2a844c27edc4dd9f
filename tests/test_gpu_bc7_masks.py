"""GPU: BC7 with some modes only.  First fits come from the modes that are on
(a 3-subset or 2-subset partition or a rotation), and with one-subset modes
alone every candidate is fitted: bit-exact against the oracle's exhaustive
search, below and above the size from which a wave takes its blocks alone."""
import numpy as np
import pytest

import oracle as O
from conftest import smooth_blocks
from test_gpu_bc7_search import _blocks, _prim_desc

MASKS = [0x01, 0x02, 0x04, 0x08, 0x10, 0x20, 0x40, 0x80, 0x05, 0x41, 0x42, 0x8A, 0x8B, 0xCB, 0x60, 0x70, 0x12, 0x29, 0x84]
KINDS = ["gradient", "near_constant", "two_level", "constant", "random"]


def _mixed(n, seed):
    t = np.concatenate([_blocks(k, n, seed)[None] for k in KINDS] + [smooth_blocks(n, seed, 3)[None]])
    return np.ascontiguousarray(np.moveaxis(t, 0, 1).reshape(-1, 16, 4)[:n])


@pytest.mark.gpu
@pytest.mark.parametrize("mask", MASKS)
def test_modes_equal_exhaustive(mask):
    import torch
    from paper_2607_14513_amd import gsbc
    nblk = 336                 # ragged: one run of 512 indices
    t = _mixed(nblk, mask)
    want, sse = O.bc7_encode(t, mode_mask=mask)
    with gsbc.Context(0) as ctx:
        out, _, s = ctx.encode(torch.from_numpy(t[None]).cuda(), _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7, want_sse=True,
                               params=gsbc.default_params(bc7_mode_mask=mask))
    assert np.array_equal(out.cpu().numpy()[:16 * nblk].reshape(-1, 16), want.reshape(-1, 16))
    assert s[1][0] == int(np.asarray(sse, np.int64).sum())


@pytest.mark.gpu
@pytest.mark.parametrize("mask", [0x01, 0x02, 0x70, 0x8A])
def test_modes_in_large_encodes(mask):
    import torch
    from paper_2607_14513_amd import gsbc
    nblk = (1 << 17) + 272
    t = np.tile(_mixed(336, mask), (-(-nblk // 336), 1, 1))[:nblk].copy()
    want, _ = O.bc7_encode(t[:336], mode_mask=mask)
    with gsbc.Context(0) as ctx:
        out, _, _ = ctx.encode(torch.from_numpy(t[None]).cuda(), _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7,
                               params=gsbc.default_params(bc7_mode_mask=mask))
    got = out.cpu().numpy()[:16 * nblk].reshape(-1, 16)
    assert np.array_equal(got, np.tile(want.reshape(-1, 16), (-(-nblk // 336), 1))[:nblk])


@pytest.mark.gpu
@pytest.mark.parametrize("mask", [0x01, 0x02, 0x04, 0x05, 0x42, 0x8A])
def test_slices_that_keep_their_candidates(mask):
    """Slices of 64 blocks that bounds rule little out of, among others, in two
    chunks of the scratch and a ragged end; partitions of one shape."""
    import torch
    from paper_2607_14513_amd import gsbc
    kinds = ["gradient", "random", "near_constant", "constant", "gradient", "two_level"]
    unit = np.concatenate([_blocks(k, 64, 40 + i) for i, k in enumerate(kinds)])
    nblk = (1 << 19) + (1 << 17) + 272
    want, _ = O.bc7_encode(unit, mode_mask=mask)
    with gsbc.Context(0) as ctx:
        tex = torch.from_numpy(unit).cuda().repeat(-(-nblk // len(unit)), 1, 1)[:nblk].contiguous()
        out, _, _ = ctx.encode(tex[None], _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7, params=gsbc.default_params(bc7_mode_mask=mask))
        ref = torch.from_numpy(want.reshape(-1, 16)).cuda().repeat(-(-nblk // len(unit)), 1)[:nblk]
        ctx.sync()
        assert torch.equal(out[:16 * nblk].view(-1, 16), ref)
