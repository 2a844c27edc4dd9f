"""The BC7 search fits only the candidates whose lower bound leaves them a
chance: bit-exact against the oracle's exhaustive search on blocks at the
edges of the bounds, of the windows of blocks and of the chunks of the scratch,
and the bounds' constants re-derived from the index weights."""
import os
import re

import numpy as np
import pytest

import oracle as O
from conftest import ROOT, random_blocks, rgba


def _blocks(kind, n, seed):
    rng = np.random.default_rng(seed)
    base = rng.integers(0, 256, (n, 1, 3))
    if kind == "gradient":        # colours along a line, little off it: most candidates stay
        x = rng.uniform(60, 200, (n, 1, 3)) + rng.normal(0, 1, (n, 1, 3)) * 40 * rng.uniform(-1, 1, (n, 16, 1))
        return rgba(np.clip(x + rng.normal(0, 2, (n, 16, 3)), 0, 255).round())
    if kind == "near_constant":   # residuals below the bounds' slack
        return rgba(np.clip(base + rng.integers(0, 2, (n, 16, 3)), 0, 255))
    if kind == "two_level":       # exact fits, ties between candidates, flat subsets
        return rgba(np.where(rng.integers(0, 2, (n, 16, 1)) == 1, base, rng.integers(0, 256, (n, 1, 3))))
    if kind == "one_channel":     # the other channels constant: degenerate scatter matrices
        x = np.broadcast_to(base, (n, 16, 3)).copy()
        c = rng.integers(0, 3, n)
        x[np.arange(n), :, c] = rng.integers(0, 256, (n, 16))
        return rgba(x)
    if kind == "constant":        # every partition of a mode ties
        return rgba(np.repeat(base, 16, 1))
    if kind == "corners":         # the largest sums and covariances
        return rgba(255 * rng.integers(0, 2, (n, 16, 3)))
    return random_blocks(n, seed)


def _prim_desc(gsbc, nblk):
    d = gsbc.StreamDesc()
    d.n_prims = d.n_pad = d.blocks_per_stream = nblk
    d.arrangement, d.n_streams = gsbc.ARR_PRIM, 1
    for k in range(16):
        d.vmin[k], d.vmax[k] = 0.0, 1.0
    return d


@pytest.mark.gpu
@pytest.mark.parametrize("kind,nblk", [("gradient", 1040), ("near_constant", 272), ("two_level", 272), ("one_channel", 272),
                                       ("corners", 272), ("constant", 272), ("random", 16), ("random", 80), ("random", 4112)])
def test_search_equals_exhaustive(kind, nblk):
    import torch
    from paper_2607_14513_amd import gsbc
    t = _blocks(kind, nblk, 11)
    want, sse = O.bc7_encode(t)
    with gsbc.Context(0) as ctx:
        out, d, s = ctx.encode(torch.from_numpy(t[None]).cuda(), _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7, want_sse=True)
    assert np.array_equal(out.cpu().numpy()[:16 * nblk].reshape(-1, 16), want.reshape(-1, 16))
    assert s[1][0] == int(np.asarray(sse, np.int64).sum())


@pytest.mark.gpu
def test_search_past_one_chunk():
    import torch
    from paper_2607_14513_amd import gsbc
    nblk = (1 << 19) + 528     # one chunk of bounds and a ragged piece of the next
    t = _blocks("random", nblk, 12)
    pick = np.r_[0:32, (1 << 19) - 32:(1 << 19) + 32, nblk - 32:nblk]
    want, _ = O.bc7_encode(t[pick])
    with gsbc.Context(0) as ctx:
        out, _, _ = ctx.encode(torch.from_numpy(t[None]).cuda(), _prim_desc(gsbc, nblk), fmt=gsbc.FMT_BC7)
    assert np.array_equal(out.cpu().numpy()[:16 * nblk].reshape(-1, 16)[pick], want.reshape(-1, 16))


def _cheb(weights):
    """Largest over D mod 64 of the minimax distance of the rounded
    interpolants' deviations from a straight line in the weight (by the
    alternation theorem: the largest over index triples)."""
    w = np.array(weights, float)
    worst = 0.0
    for D in range(64):
        e = np.floor((w * D + 32) / 64) - w * D / 64
        for i in range(len(w)):
            for j in range(i + 1, len(w)):
                for k in range(j + 1, len(w)):
                    a = (w[k] - w[j]) / (w[k] - w[i])
                    worst = max(worst, abs(a * e[i] + (1 - a) * e[k] - e[j]) / 2)
    return worst


def test_bound_slack_covers_rounded_palettes():
    src = open(os.path.join(ROOT, "paper_2607_14513_amd", "csrc", "bc7_encode.hip")).read()
    slack = {m: float(v) for m, v in re.findall(r"(kSlack\w+) = ([0-9.]+)f", src)}
    for nb in (2, 3, 4):
        c = _cheb([(128 * i + 2 ** nb - 1) // (2 * (2 ** nb - 1)) for i in range(2 ** nb)])
        assert 3 ** 0.5 * c <= slack[f"kSlack{nb}"] < 3 ** 0.5 * c + 0.002
        if nb == 3:
            assert 2 ** 0.5 * c <= slack["kSlackRot"] < 2 ** 0.5 * c + 0.002
