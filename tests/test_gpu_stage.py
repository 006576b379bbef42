"""Rescan with the map staged through LDS against the FP64 oracle and the plain form.

DST_UNBIN_BPW=16 stages the map values of sixteen baselines, up to 10112 doubles
(three, two or one per pixel); a block on more pixels than that reads them from
memory.  Bars as for the plain form.
"""
import numpy as np
import pytest

from oracle import destripe as O
from problems import args, toy

pytestmark = pytest.mark.gpu


def rel(a, b):
    a, b = np.asarray(a, float), np.asarray(b, float)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def context(monkeypatch, staged):
    from paper_1309_5609_amd import dst
    monkeypatch.setenv("DST_UNBIN_BPW", "16" if staged else "4")
    return dst.Context(0)


@pytest.mark.parametrize("name", ["plain", "masked", "unequal", "QU", "T", "IQU"])
def test_staged_against_the_oracle(monkeypatch, name):
    from paper_1309_5609_amd import dst
    p = toy(**{"plain": {}, "masked": dict(mask_fraction=0.07), "unequal": dict(weights=(2.0e6, 5.0e6, 0.7e6)),
               "QU": dict(streams="QU"), "T": dict(streams="T"),
               "IQU": dict(streams="IQU", n_samples=20000, L=400)}[name])
    c = context(monkeypatch, True)
    dp = dst.to_device(p)
    out = dst.dst_solve(c, dp, tol=1e-13, max_iter=3000)
    eager = dst.dst_solve(c, dp, tol=1e-13, max_iter=3000, flags=dst.DST_SOLVE_NO_GRAPH)
    ref = O.solve(*args(p), tol=1e-13, max_iter=3000)
    assert abs(out["iterations"] - ref.iterations) <= 1 + ref.iterations // 50
    assert rel(out["baselines"].cpu().numpy(), ref.baselines) < 1e-9
    ok = {"QU": ref.valid_QU}.get(p.streams, ref.valid_T)
    assert rel(out["destriped_map"].cpu().numpy()[ok], ref.destriped_map[ok]) < 1e-9
    for k in ("baselines", "destriped_map"):
        assert np.array_equal(out[k].cpu().numpy(), eager[k].cpu().numpy())
    c.close()


# baselines: one, a full block, one more, past eight blocks; lists that fit and that do not (long baselines on fine
# pixels), and blocks of both kinds (masked: the first third of the samples)
@pytest.mark.parametrize("streams,dtype", [("T", "float64"), ("T", "float32"), ("QU", "float64"), ("TQU", "float32"),
                                           ("TQU", "float64")])
@pytest.mark.parametrize("n,L,nside", [(50, 50, 4), (16 * 7, 7, 2), (16 * 7 + 1, 7, 8), (16 * 129 * 5, 5, 8),
                                       (120000, 1500, 128), (120000, 300, 64)])
def test_staged_against_plain(monkeypatch, streams, dtype, n, L, nside):
    from paper_1309_5609_amd import dst
    p = toy(n_samples=n, L=L, nside=nside, streams=streams)
    if n >= 10000:
        p.pix[: n // 3][np.arange(n // 3) % 64 != 0] = -1
    dp = dst.to_device(p, tod_dtype=dtype, psi_dtype=dtype)
    res = []
    for staged in (True, False):
        c = context(monkeypatch, staged)
        res.append(dst.dst_solve(c, dp, tol=1e-30, max_iter=2))
        c.close()
    for k in ("baselines", "destriped_map", "binned_map"):
        # three operator applications of sums of up to n terms: n eps = 3e-11
        assert rel(res[0][k].cpu().numpy(), res[1][k].cpu().numpy()) < 1e-10, k


def test_staged_group(monkeypatch):
    """Channels advanced together, their rescans staged; several stream sets, one of them (a radiometer) never staged."""
    from paper_1309_5609_amd import dst
    ps = [toy(n_samples=9100, L=250, nside=16), toy(n_samples=30001, L=11, nside=16), toy(n_samples=700, L=7),
          toy(streams="T"), toy(streams="T", n_samples=120000, L=1500, nside=128), toy(streams="QU"),
          toy(streams="IQU", n_samples=20000, L=400)]
    c = context(monkeypatch, True)
    dps = [dst.to_device(p) for p in ps]
    _, res = dst.dst_solve_batched(c, dps, tol=1e-13, max_iter=3000)
    _, eager = dst.dst_solve_batched(c, dps, tol=1e-13, max_iter=3000, flags=dst.DST_SOLVE_NO_GRAPH)
    for p, out, one in zip(ps, res, eager):
        ref = O.solve(*args(p), tol=1e-13, max_iter=3000)
        assert abs(out["iterations"] - ref.iterations) <= 1 + ref.iterations // 50
        assert rel(out["baselines"].cpu().numpy(), ref.baselines) < 1e-9
        ok = {"QU": ref.valid_QU}.get(p.streams, ref.valid_T)
        assert rel(out["destriped_map"].cpu().numpy()[ok], ref.destriped_map[ok]) < 1e-9
        assert np.array_equal(out["baselines"].cpu().numpy(), one["baselines"].cpu().numpy())
    c.close()
