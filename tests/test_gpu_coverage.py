"""GPU: the coverage range at sizes about the histogram's steps of 32
primitives, its 16-wave workgroups and its 256 workgroups, against the
oracle's selection of the same rank, bit for bit."""
import numpy as np
import pytest

import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opacity", [False, True])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 511, 513, 8_193, 131_073, 140_001])
def test_coverage_range(n, opacity):
    from paper_2607_14513_amd import gsbc
    rng = np.random.default_rng(n)
    # magnitudes over many exponents, with ties, zeros of both signs and a band of one value
    sh = (rng.normal(size=(n, 16, 3)) * np.exp(rng.normal(size=(n, 16, 1)) * 3)).astype(np.float32)
    sh[rng.random((n, 16, 3)) < 0.2] = -0.0
    sh[:, 5] = np.round(sh[:, 5])
    sh[:, 7] = -0.25
    mu = rng.random(n).astype(np.float32) if opacity else None
    pos = rng.random((n, 3)).astype(np.float32)
    with gsbc.Context(0) as ctx:
        d = ctx.reorder(torch.from_numpy(pos).cuda(), torch.from_numpy(sh).cuda(),
                        opacity=torch.from_numpy(mu).cuda() if opacity else None,
                        params=gsbc.default_params(quantiser=1))[2]
        lo, hi = d.ranges()
    rlo, rhi = O.band_range_coverage(O.premultiply(sh, mu) if opacity else sh)
    assert np.array_equal(np.asarray(lo, np.float32).view(np.uint32), np.asarray(rlo, np.float32).view(np.uint32))
    assert np.array_equal(np.asarray(hi, np.float32).view(np.uint32), np.asarray(rhi, np.float32).view(np.uint32))
