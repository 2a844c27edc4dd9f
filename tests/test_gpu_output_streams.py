"""GPU: outputs come from the pool of the stream that writes them, whatever
stream is torch's current one, and are kept from being written again while that
one may still read them."""
import pytest

from paper_2607_14513_amd import synth
from test_gpu_two_contexts import _scene

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SLEEP = 100_000_000   # cycles: some 50 ms


def test_contexts_on_streams_of_the_caller():
    """A dropped output does not become another context's, nor a torch
    tensor's of the current stream, while its kernel may still write it."""
    from paper_2607_14513_amd import gsbc
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    dirs = torch.from_numpy(synth.make_dirs(64, seed=7)).cuda()
    torch.cuda.synchronize()
    with gsbc.Context(0, stream=sa) as a, gsbc.Context(0, stream=sb) as b:
        xa, xb = _scene(a, gsbc, 20_011, 5), _scene(b, gsbc, 20_011, 6)
        torch.cuda.synchronize()
        ref = b.decode_eval(*xb, dirs)
        b.sync()
        ref = ref.clone()
        torch.cuda.synchronize()
        for _ in range(4):
            p = a.decode_eval(*xa, dirs).data_ptr()   # dropped at once, its kernel still running
            t = torch.empty_like(ref)
            out = b.decode_eval(*xb, dirs)
            assert p not in (out.data_ptr(), t.data_ptr())
            b.sync()
            assert torch.equal(out, ref)
        torch.cuda.synchronize()


@pytest.mark.parametrize("own", [True, False])
def test_output_read_on_another_stream(own):
    """An output made and read under stream t, dropped while t still reads."""
    from paper_2607_14513_amd import gsbc
    t, s = torch.cuda.Stream(), None if own else torch.cuda.Stream()
    d0, d1 = (torch.from_numpy(synth.make_dirs(64, seed=k)).cuda() for k in (8, 9))
    torch.cuda.synchronize()
    with gsbc.Context(0, stream=s) as ctx:
        x = _scene(ctx, gsbc, 20_011, 5)
        torch.cuda.synchronize()
        ref = ctx.decode_eval(*x, d0)
        ctx.sync()
        ref = ref.cpu()
        with torch.cuda.stream(t):
            out = ctx.decode_eval(*x, d0)
            ctx.sync()
            torch.cuda._sleep(SLEEP)
            got = out.clone()
        p = out.data_ptr()
        del out
        again = ctx.decode_eval(*x, d1)
        assert again.data_ptr() != p
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), ref)


def test_streams_of_living_outputs():
    """More contexts than the spare streams, closed while their outputs live:
    no stream is destroyed before its outputs are gone."""
    from paper_2607_14513_amd import gsbc
    dirs = torch.from_numpy(synth.make_dirs(3, seed=8)).cuda()
    many = [gsbc.Context(0) for _ in range(gsbc._SPARE_STREAMS + 3)]
    x = _scene(many[0], gsbc, 1_003, 9)
    outs = {c._own: c.decode_eval(*x, dirs) for c in many}
    for c in many:
        c.close()
    assert set(outs) <= set(gsbc._spare_streams[0]) | set(gsbc._held_streams[0])
    assert gsbc._held_streams[0] and set(gsbc._held_streams[0]) <= gsbc._pools_alive(0)
    ref = outs.popitem()[1].cpu()
    assert all(torch.equal(o.cpu(), ref) for o in outs.values())
    held = set(gsbc._held_streams[0])
    del outs, x
    more = [gsbc.Context(0) for _ in range(gsbc._SPARE_STREAMS)]   # the spare ones
    for c in more + [gsbc.Context(0)]:
        c.close()
    assert held and not held & set(gsbc._held_streams[0]) - gsbc._pools_alive(0)


def test_stream_of_another_kind():
    """Anything with a `cuda_stream` serves as a stream; outputs then come from the current stream's pool."""
    from paper_2607_14513_amd import gsbc
    st = torch.cuda.Stream()
    handle = type("Handle", (), {"cuda_stream": st.cuda_stream})()
    with torch.cuda.stream(st):
        dirs = torch.from_numpy(synth.make_dirs(3, seed=8)).cuda()
        with gsbc.Context(0, stream=handle) as ctx:
            out = ctx.decode_eval(*_scene(ctx, gsbc, 1_003, 9), dirs)
            ctx.sync()
    assert out.shape == (3, 1_003, 3)
