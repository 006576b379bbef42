"""Pixels with many more runs than the others, swept by a whole wavefront, against the FP64 oracle.

In the per-pixel setup from 16 steps of 8 or 32 lanes with four runs each on (512
or 2048 runs; not for radiometers), in the LDS and pipelined binning from 16
steps of the pixel's lanes (256 runs and up).  Bars as for the plain forms.
"""
import numpy as np
import pytest

from oracle import destripe as O
from problems import args, toy

pytestmark = pytest.mark.gpu


def rel(a, b):
    a, b = np.asarray(a, float), np.asarray(b, float)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def deep(runs, nside, streams, **kw):
    """Every other sample of the first 2 * runs on one pixel, one run each, and another pixel with half as many."""
    p = toy(n_samples=12000, L=250, nside=nside, streams=streams, **kw)
    p.pix[: 2 * runs : 2] = 5
    p.pix[2 * runs : 3 * runs : 2] = 11
    p.pix[1 : 2 * runs : 2][p.pix[1 : 2 * runs : 2] == 5] = 6
    return p


@pytest.mark.parametrize("form", ["0", "1", "2"])
@pytest.mark.parametrize("streams,weights", [("T", (2.0e6,) * 3), ("QU", (2.0e6,) * 3), ("TQU", (2.0e6, 5.0e6, 0.7e6)),
                                             ("IQU", (2.0e6,) * 3)])
@pytest.mark.parametrize("nside,runs", [(16, 255), (16, 257), (16, 511), (16, 512), (16, 513), (16, 3700), (2, 2047),
                                        (2, 2049)])
def test_deep_pixels(monkeypatch, nside, runs, streams, weights, form):
    from paper_1309_5609_amd import dst
    monkeypatch.setenv("DST_BIN_FORM", form)
    p = deep(runs, nside, streams, weights=weights)
    other = deep(runs // 2, nside, streams, weights=weights, cfg=301)
    c = dst.Context(0)
    alone = dst.dst_solve(c, dst.to_device(p), tol=1e-13, max_iter=3000)
    group = dst.dst_solve_batched(c, [dst.to_device(p), dst.to_device(other)], tol=1e-13, max_iter=3000)[1]
    for q, out in ((p, alone), (p, group[0]), (other, group[1])):
        ref = O.solve(*args(q), tol=1e-13, max_iter=3000)
        assert np.array_equal(out["hits"].cpu().numpy(), ref.hits)
        assert rel(out["baselines"].cpu().numpy(), ref.baselines) < 1e-9
        ok = {"QU": ref.valid_QU}.get(streams, ref.valid_T)
        assert rel(out["binned_map"].cpu().numpy()[ok], ref.binned_map[ok]) < 1e-9
        assert rel(out["destriped_map"].cpu().numpy()[ok], ref.destriped_map[ok]) < 1e-9
    c.close()
