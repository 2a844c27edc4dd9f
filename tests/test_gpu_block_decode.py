"""GPU: whole-block decoding.  Random blocks of every BC7 mode (the reserved
one too) and of BC1 decode to the oracle's texels byte for byte at sizes about
the 256-block and 256-slot tiles, and evaluating all slots (whole blocks,
handed over in LDS) gives the bits of evaluating the same slots as a list
(texel by texel), in every arrangement and with dropped bands."""
import numpy as np
import pytest

import oracle as O
from paper_2607_14513_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [1, 16, 255, 256, 257, 1_003, 4_111, 8_193]


def _coded(gsbc, n, arrangement, streams, seed):
    """Payload and descriptor of random blocks; stream formats vary."""
    rng = np.random.default_rng(seed)
    d = gsbc.StreamDesc()
    npad = (n + 15) // 16 * 16
    nblk = {0: npad // 16, 1: npad, 2: npad // 4}[arrangement]
    parts, pos = [], 0
    for k in range(streams):
        f = int(rng.choice([gsbc.FMT_BC7, gsbc.FMT_BC7, gsbc.FMT_BC1] + ([gsbc.FMT_NONE] if arrangement == 0 and k else [])))
        size = {gsbc.FMT_BC7: 16, gsbc.FMT_BC1: 8, gsbc.FMT_NONE: 0}[f]
        b = rng.integers(0, 256, (nblk, size), dtype=np.uint8)
        if f == gsbc.FMT_BC7:
            m = rng.integers(0, 9, nblk)
            b[:, 0] = np.where(m < 8, (b[:, 0].astype(int) & ~((2 << m) - 1)) | (1 << m), 0).astype(np.uint8)
            b[rng.random(nblk) < 0.1, 1:] = 255
        d.format[k], d.offset[k] = f, pos
        raw = b.reshape(-1)
        parts += [raw, np.zeros(-raw.size % 16, np.uint8)]
        pos += raw.size + (-raw.size % 16)
    for k in range(16):
        d.vmin[k], d.vmax[k] = -0.3 - 0.05 * k, 0.9 - 0.03 * k
    d.n_prims, d.n_pad, d.blocks_per_stream, d.payload_bytes = n, npad, nblk, pos
    d.arrangement, d.n_streams = arrangement, streams
    return np.concatenate(parts + [np.zeros(16, np.uint8)])[:max(pos, 16)], d


@pytest.mark.parametrize("arrangement,streams", [(0, 16), (0, 4), (0, 1), (1, 1), (2, 4), (2, 1)])
def test_blocks(arrangement, streams):
    from paper_2607_14513_amd import gsbc
    with gsbc.Context(0) as ctx:
        for n in SIZES:
            payload, d = _coded(gsbc, n, arrangement, streams, 1000 * arrangement + 10 * streams + n)
            blocks = torch.from_numpy(payload).cuda()
            tex = ctx.decode(blocks, d).cpu().numpy()
            for k in range(streams):
                if d.format[k] == gsbc.FMT_NONE:
                    assert not tex[k].any()
                    continue
                size = 16 if d.format[k] == gsbc.FMT_BC7 else 8
                raw = payload[d.offset[k]:d.offset[k] + size * tex.shape[1]].reshape(-1, size)
                ref = (O.bc7_decode if size == 16 else O.bc1_decode)(raw)
                assert np.array_equal(tex[k].reshape(ref.shape), ref), (n, k)
            slots = torch.arange(n, dtype=torch.int32, device="cuda")
            for V in (3, 300):
                dirs = torch.from_numpy(synth.make_dirs(V, seed=n)).cuda()
                assert torch.equal(ctx.decode_eval(blocks, d, dirs), ctx.decode_eval(blocks, d, dirs, prim_idx=slots)), (n, V)
            pos = torch.from_numpy(np.random.default_rng(n).normal(size=(n, 3)).astype(np.float32)).cuda()
            perm = torch.randperm(n, device="cuda").to(torch.int32)
            view = (0.3, -2.0, 1.5)
            assert torch.equal(ctx.decode_eval_view(blocks, d, pos, perm, view),
                               ctx.decode_eval_view(blocks, d, pos, perm, view, prim_idx=slots)), n
