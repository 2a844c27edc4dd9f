"""GPU: what slots that no tile lists hold does not matter to blend_tiles.  Their
perm entries may name no primitive, their primitives' positions and blocks may
hold anything, on the route that computes the colours first too, which a list
buffer longer than the entries in use also takes; the image is that of the
whole scene bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_blend_routes import VIEW, _inputs, dev   # noqa: E402


def _spoilt(blocks, d, pos, perm, used, n):
    """The scene with all that belongs to unlisted slots only made unusable."""
    off = np.setdiff1d(np.arange(n), used)
    p = perm.cpu().numpy().copy()
    xyz = pos.cpu().numpy().copy()
    xyz[p[off]] = np.nan
    p[off] = -1
    per = {0: 16, 1: 1, 2: 4}[d.arrangement]               # slots a block
    size = np.array([16 if f == 7 else 8 for f in d.formats()])
    raw = blocks.cpu().numpy().copy()
    gone = np.setdiff1d(np.arange(d.blocks_per_stream), used // per)
    for k in range(d.n_streams):
        o = int(d.offset[k])
        raw[o:o + size[k] * d.blocks_per_stream].reshape(-1, size[k])[gone] = 0xA5
    return dev(raw), dev(xyz), dev(p)


@pytest.mark.parametrize("n,arrangement", [(257, 0), (4_111, 1), (4_111, 2), (20_011, 0)])
@pytest.mark.parametrize("share", [0.9, 0.05])
def test_only_listed_slots_are_read(n, arrangement, share):
    from paper_2607_14513_amd import gsbc
    tx, ty = 6, 4
    with gsbc.Context(0) as ctx:
        blocks, d, pos, perm, mu, foot, ts, lst = _inputs(ctx, gsbc, n, tx, ty, 21, arrangement)
        used = np.flatnonzero(np.random.default_rng(22).random(n) < share)   # the slots that may be listed
        keep = np.isin(lst, used)
        cnt = np.add.reduceat(np.r_[keep.astype(np.int64), 0], ts[:-1]) * (np.diff(ts) > 0)
        lst, ts = lst[keep], np.r_[0, np.cumsum(cnt)].astype(np.int32)
        assert ts[-1] == lst.size
        lst = np.concatenate([lst, np.full(1 << 15, 7, np.int32)])           # the buffer's unused end
        tail = (mu, foot, dev(ts), dev(lst), tx, ty)
        img, T = ctx.blend_tiles(blocks, d, pos, perm, VIEW, *tail)
        colours = ctx.decode_eval_view(blocks, d, pos, perm, VIEW)
        ref, refT = ctx.blend_tiles_colours(colours, perm, *tail)
        raw, xyz, p = _spoilt(blocks, d, pos, perm, np.unique(lst[:ts[-1]]), n)
        got, gotT = ctx.blend_tiles(raw, d, xyz, p, VIEW, *tail)
        ctx.sync()
    for a, b in ((img, ref), (T, refT), (got, ref), (gotT, refT)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("rows", ["own", "more"])
def test_all_slots_or_marked_ones(rows):
    """Long lists over a scene whose perm names its own primitives (every slot is
    decoded) and over a part of a larger set (perm beyond n_prims: the listed
    ones only), in turn on one context."""
    from paper_2607_14513_amd import gsbc
    n, tx, ty = 20_011, 6, 4
    with gsbc.Context(0) as ctx:
        blocks, d, pos, perm, mu, foot, ts, lst = _inputs(ctx, gsbc, n, tx, ty, 23, 0)
        lst = np.concatenate([lst, np.full(1 << 15, 7, np.int32)])
        if rows == "more":          # the same primitives behind n others
            pos, mu, foot = (torch.cat([torch.full_like(t, float("nan")), t]) for t in (pos, mu, foot))
            perm = perm + n
        tail = (mu, foot, dev(ts.astype(np.int32)), dev(lst), tx, ty)
        colours = ctx.decode_eval_view(blocks, d, pos, perm, VIEW)
        ref, refT = ctx.blend_tiles_colours(colours, perm, *tail)
        used = np.unique(lst[:ts[-1]])
        off = np.setdiff1d(np.arange(n), used)
        wild = perm.clone()
        wild[torch.from_numpy(off).cuda()] = 0x7FFFFFFF
        for p in (perm, wild, perm):
            got, gotT = ctx.blend_tiles(blocks, d, pos, p, VIEW, *tail)
            assert torch.equal(got.view(torch.int32), ref.view(torch.int32))
            assert torch.equal(gotT.view(torch.int32), refT.view(torch.int32))
