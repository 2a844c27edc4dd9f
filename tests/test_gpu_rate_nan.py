"""GPU: the band choice with gains that are infinite or no number (a band whose
range is) follows the oracle's rule, which picks the bands one by one."""
import numpy as np
import pytest

import oracle as O
from conftest import smooth_blocks

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

INF, NAN = np.float32(np.inf), np.float32(np.nan)
CASES = {"nan first": {1: NAN}, "nan between": {4: NAN, 11: NAN}, "nan last": {15: NAN}, "infinite": {3: INF, 9: INF},
         "all nan": {k: NAN for k in range(1, 16)}, "both": {2: INF, 6: NAN, 7: INF, 12: NAN}}


@pytest.mark.parametrize("case", list(CASES))
def test_choice_with_gains_that_are_no_numbers(case):
    from paper_2607_14513_amd import gsbc
    nblk = 17
    tex = np.stack([smooth_blocks(nblk, 300 + k, spread=2 + 3 * ((5 * k) % 16)) for k in range(16)])
    tex[9] = tex[9, :, :1]                       # one colour a block: both formats may be exact
    tex[9, :, :, :3] = 0
    d = gsbc.StreamDesc()
    d.n_prims = d.n_pad = 16 * nblk
    d.blocks_per_stream, d.arrangement, d.n_streams = nblk, gsbc.ARR_BANDS, 16
    for k in range(16):
        d.vmin[k], d.vmax[k] = -0.4 - 0.02 * k, 0.5 + 0.03 * ((7 * k) % 16)
    for k, v in CASES[case].items():
        d.vmax[k] = v
    vmin, vmax = d.ranges()
    with gsbc.Context(0) as ctx:
        t = torch.from_numpy(tex).cuda()
        for rate in (4.25, 4.5, 5.25, 6.0, 7.5, 7.75, 8.0):
            _, d2, sse = ctx.encode(t, d, fmt=gsbc.FMT_AUTO, rate=rate, want_sse=True)
            want = O.rate_select(sse[0], sse[1], vmin, vmax, rate)
            assert np.array_equal(d2.formats(), want), rate
