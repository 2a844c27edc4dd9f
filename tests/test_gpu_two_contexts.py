"""GPU: contexts on torch's default stream.  Each works on a stream of its
own, so an output dropped by the caller while its kernel still runs must not
become another context's output; closed contexts hand their streams on and
keep few of them."""
import numpy as np
import pytest

from paper_2607_14513_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _scene(ctx, gsbc, n, seed):
    pos, sh = synth.make_scene(n, seed=seed)
    _, tex, d = ctx.reorder(torch.from_numpy(pos).cuda(), torch.from_numpy(sh).cuda())
    blocks, d2, _ = ctx.encode(tex, d, fmt=gsbc.FMT_BC7)
    return blocks, d2


def test_dropped_output_is_not_handed_to_another_context():
    from paper_2607_14513_amd import gsbc
    with gsbc.Context(0) as a, gsbc.Context(0) as b:
        sa, sb = _scene(a, gsbc, 20_011, 5), _scene(b, gsbc, 20_011, 6)
        dirs = torch.from_numpy(synth.make_dirs(64, seed=7)).cuda()
        ref = b.decode_eval(*sb, dirs).clone()
        for _ in range(6):
            p = a.decode_eval(*sa, dirs).data_ptr()   # dropped at once, its kernel still running
            out = b.decode_eval(*sb, dirs)
            assert out.data_ptr() != p
            assert torch.equal(out, ref)


def test_streams_of_closed_contexts():
    from paper_2607_14513_amd import gsbc
    dirs = torch.from_numpy(synth.make_dirs(3, seed=8)).cuda()
    with gsbc.Context(0) as c:
        scene = _scene(c, gsbc, 1_003, 9)
        ref = c.decode_eval(*scene, dirs).cpu().numpy()
    many = [gsbc.Context(0) for _ in range(12)]
    assert len({c._own for c in many}) == 12
    outs = [c.decode_eval(*scene, dirs) for c in many]
    for c in many:
        c.close()
    assert len(gsbc._spare_streams[0]) <= 8
    assert all(np.array_equal(o.cpu().numpy(), ref) for o in outs)
