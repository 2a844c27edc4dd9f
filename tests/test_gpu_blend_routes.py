"""GPU: the two routes of blend_tiles.  Lists of at least one entry per four
slots have every slot's colour computed first, shorter ones are decoded entry
by entry; a capture whose scratch has no room for the colours takes the second
route too.  All give the same image and transmittance bit for bit."""
import numpy as np
import pytest

from paper_2607_14513_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

VIEW = (0.5, 0.45, 2.5)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _inputs(ctx, gsbc, n, tx, ty, seed, arrangement=0):
    pos, sh = synth.make_scene(n, seed=seed)
    p = gsbc.default_params(arrangement=arrangement)
    perm, tex, d = ctx.reorder(dev(pos), dev(sh), params=p)
    blocks, d2, _ = ctx.encode(tex, d, fmt=gsbc.FMT_BC7)
    foot, ts, lst = synth.make_tiles(pos, VIEW, tx, ty, seed=seed)
    slot = np.argsort(perm.cpu().numpy().view(np.uint32)).astype(np.int32)
    return blocks, d2, dev(pos), perm, dev(synth.make_opacity(n, seed=seed)), dev(foot), ts.astype(np.int64), slot[lst]


def _shorter(ts, lst, most):
    """The first entries of each tile's list, `most` in all at the most."""
    keep = max(1, most // (len(ts) - 1))
    cnt = np.minimum(np.diff(ts), keep)
    out = np.concatenate([lst[a:a + c] for a, c in zip(ts[:-1], cnt)])
    return np.concatenate([[0], np.cumsum(cnt)]), out


@pytest.mark.parametrize("n,arrangement", [(257, 0), (3_001, 0), (20_011, 1), (20_011, 2)])
def test_short_and_padded_lists(n, arrangement):
    from paper_2607_14513_amd import gsbc
    with gsbc.Context(0) as ctx:
        blocks, d, pos, perm, mu, foot, ts, lst = _inputs(ctx, gsbc, n, 5, 4, 11, arrangement)
        ts, lst = _shorter(ts, lst, n // 4)
        assert len(lst) <= n // 4
        args = (blocks, d, pos, perm, VIEW, mu, foot, dev(ts.astype(np.int32)))
        for bad in (False, True):
            if bad:
                lst = lst.copy()
                lst[len(lst) // 2] = n + 2                      # past the scene: NaN
            img, T = ctx.blend_tiles(*args, dev(lst), 5, 4)
            # entries that no tile uses make the list long enough for the other route
            img2, T2 = ctx.blend_tiles(*args, dev(np.concatenate([lst, np.zeros(n, np.int32)])), 5, 4)
            assert torch.equal(img.view(torch.int32), img2.view(torch.int32))
            assert torch.equal(T.view(torch.int32), T2.view(torch.int32))


def test_captured_without_room():
    """Replayed several times with eager work between: the capture decodes the
    entries in the blend where the context's scratch has no room."""
    from paper_2607_14513_amd import gsbc
    n, tx, ty = 100_003, 6, 5
    with gsbc.Context(0) as c0:
        inputs = _inputs(c0, gsbc, n, tx, ty, 12)
    blocks, d, pos, perm, mu, foot, ts, lst = inputs
    lst = np.concatenate([lst, np.zeros(n, np.int32)])
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with gsbc.Context(0, stream=stream) as ctx, torch.cuda.stream(stream):
        args = (blocks, d, pos, perm, VIEW, mu, foot, dev(ts.astype(np.int32)))
        short = dev(lst[:1])
        ctx.blend_tiles(*args[:-1], torch.zeros(tx * ty + 1, dtype=torch.int32, device="cuda"), short, tx, ty)
        before = ctx.arena_info()
        assert before[0] < 12 * n
        ld = dev(lst)
        img = torch.empty((16 * ty, 16 * tx, 3), dtype=torch.float32, device="cuda")
        T = torch.empty((16 * ty, 16 * tx), dtype=torch.float32, device="cuda")
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            ctx.blend_tiles(*args, ld, tx, ty, image=img, transmittance=T)
        assert ctx.arena_info() == before
        ref, refT = ctx.blend_tiles(*args, ld, tx, ty)          # eager: colours first
        assert ctx.arena_info()[0] >= 12 * n
        for _ in range(3):
            img.zero_()
            T.zero_()
            g.replay()
            stream.synchronize()
            assert torch.equal(img, ref) and torch.equal(T, refT)
            ctx.decode_eval_view(blocks, d, pos, perm, VIEW)
        stream.synchronize()
