"""The bucket form on coarse maps and long stays on a pixel, against the atomic form.

Small maps deal fewer pixels at a time and keep up to 64 copies of a pixel's sums
(map sizes at the edges of both); where a wavefront's lanes stay on one pixel,
their stretch is one record.  Bounds as for the bucket form's other tests.
"""
import numpy as np
import pytest

from test_gpu_bucket import BEYOND, EPS

pytestmark = pytest.mark.gpu


def timeline(n, n_pix, pattern, streams, dtype):
    import torch
    rng = np.random.default_rng([n, n_pix])
    if pattern == "stay":  # stays of 1 to 2000 samples
        pix = np.repeat(rng.integers(0, n_pix, n), rng.integers(1, 3, n) ** rng.integers(1, 12, n))[:n]
    elif pattern == "edges":  # stays about a lane's, half a wavefront's and a wavefront's 4, 128 and 256 samples
        pix = np.repeat(rng.integers(0, n_pix, n), rng.choice([3, 4, 5, 127, 128, 129, 255, 256, 257, 300], n))[:n]
    else:
        pix = rng.integers(0, n_pix, n)
    pix = pix.astype(np.int32)
    if pattern == "edges":
        pix[rng.random(n) < 0.002] = -1
    psi = rng.uniform(-3.0, 3.0, n)
    tod = rng.standard_normal(({"T": 1, "QU": 2, "TQU": 3}[streams], n))
    return (torch.from_numpy(pix).cuda(), None if streams == "T" else torch.from_numpy(psi).to(dtype).cuda(),
            torch.from_numpy(tod).to(dtype).cuda())


@pytest.mark.parametrize("n_pix", [1, 5, 255, 256, 257, 511, 513, 3000, 16383, 16385, 200_001])
@pytest.mark.parametrize("pattern", ["stay", "edges", "random"])
@pytest.mark.parametrize("streams,weights,dtype", [("T", (2.0, 1.0, 1.0), "float32"), ("TQU", (2.0, 3.0, 3.0), "float64"),
                                                   ("QU", (1.0, 3.0, 0.5), "float32")])
def test_coarse(streams, weights, dtype, pattern, n_pix):
    import torch
    from paper_1309_5609_amd import dst
    c = dst.Context(0)
    n, L = 40_007, 300
    arrays = timeline(n, n_pix, pattern, streams, getattr(torch, dtype))
    bad = None
    if n_pix > 5 and streams != "T":  # an angle that is no number leaves its pixel's q/u block invalid
        arrays[1][n // 3] = float("nan")
        bad = int(arrays[0][n // 3])
    base = torch.from_numpy(np.random.default_rng(3).standard_normal((arrays[2].shape[0], -(-n // L)))).cuda()
    res = []
    for pix in (n_pix, BEYOND):
        p = dst.Problem(*arrays, pix, L, streams, weights)
        hits, blk, valid = dst.dst_pixel_setup(c, p)
        s, hits2 = dst.dst_bin(c, p, baselines=base)
        m, _ = dst.dst_bin(c, p, as_map=True)
        dst.dst_synchronize(c)
        res.append([x[:n_pix].cpu().numpy() for x in (hits, blk, valid, s, hits2, m)])
    (h, blk, v, s, h2, m), (rh, rblk, rv, rs, _, rm) = res
    assert np.array_equal(h, rh) and np.array_equal(h2, rh) and np.array_equal(v, rv)
    assert h.sum() == int((arrays[0] >= 0).sum())
    if bad is not None and bad >= 0:
        assert not v[bad] & 2
    hh, w = h[:, None] + 8.0, max(weights)
    assert np.array_equal(np.isnan(blk), np.isnan(rblk))
    assert np.all(np.nan_to_num(np.abs(blk - rblk)) <= EPS * hh * h[:, None] * w)
    x = 2.0 * float(arrays[2].abs().max() + base.abs().max())
    assert np.all(np.abs(s - rs) <= EPS * hh * h[:, None] * w * x)
    assert np.all(np.abs(m - rm) <= EPS * hh * x * 4.0 * w / min(weights))
    c.close()


@pytest.mark.parametrize("weights", [(1.0, 3.0, 3.0), (1.0, 3.0, 2.0)])
@pytest.mark.parametrize("n_pix", [1, 48, 700])
def test_coarse_in_pieces(n_pix, weights):
    """Sums carried from piece to piece: a captured call on a timeline longer than the workspace it finds."""
    import torch
    from paper_1309_5609_amd import dst
    n = 1_300_001
    c, e = dst.Context(0), dst.Context(0)
    p = dst.Problem(*timeline(n, n_pix, "stay", "TQU", torch.float64), n_pix, 300, "TQU", weights)
    short = dst.Problem(*(x[..., :999].contiguous() for x in (p.pix, p.psi, p.tod)), n_pix, 300, "TQU", weights)
    dst.dst_bin(c, short)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        got, hits = dst.dst_bin(c, p)
    for k in range(3):
        p.tod.mul_(-1.5)
        want, want_hits = dst.dst_bin(e, p)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(hits, want_hits)
        h = want_hits.double()[:, None]
        assert bool(((got - want).abs() <= EPS * (h + 8.0) * h * 6.0 * float(p.tod.abs().max())).all())
    c.close()
    e.close()
