"""The other forms of the iterations' binning (baseline values in LDS; pipelined gathers) against the FP64 oracle.

DST_BIN_FORM=1 keeps the baseline values in LDS wherever they fit (20224
doubles: 20224 baselines of one stream, 10112 of q/u, 6741 of T/q/u),
DST_BIN_FORM=2 gathers them in the pipelined form wherever there are q/u
streams, 0 is the plain form.  Bars as for the plain form: baselines and maps
within 1e-9 of the oracle at tolerance 1e-13, equal iteration counts (+-1),
graph replay with the bits of launches one by one.
"""
import numpy as np
import pytest

from oracle import destripe as O
from problems import args, toy

pytestmark = pytest.mark.gpu


def rel(a, b):
    a, b = np.asarray(a, float), np.asarray(b, float)
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def context(monkeypatch, form):
    from paper_1309_5609_amd import dst
    monkeypatch.setenv("DST_BIN_FORM", str(form))
    return dst.Context(0)


VARIANTS = {
    "plain": dict(),
    "masked": dict(mask_fraction=0.07),
    "unequal": dict(weights=(2.0e6, 5.0e6, 0.7e6)),
    "QU": dict(streams="QU"),
    "T": dict(streams="T"),
    "IQU": dict(streams="IQU", n_samples=20000, L=400),
    "fewpix": dict(nside=1, n_samples=200000, L=50),  # thousands of runs per pixel
    "finepix": dict(nside=64, n_samples=30000, L=300),  # one or two runs per pixel
}


@pytest.mark.parametrize("form", [1, 2])
@pytest.mark.parametrize("name", list(VARIANTS))
def test_form(monkeypatch, name, form):
    from paper_1309_5609_amd import dst
    p = toy(**VARIANTS[name])
    c = context(monkeypatch, form)
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


@pytest.mark.parametrize("form", [1, 2])
@pytest.mark.parametrize("streams,n,dtype", [("T", 20224, "float64"), ("T", 20225, "float64"), ("QU", 10112, "float32"),
                                             ("QU", 10113, "float64"), ("TQU", 6741, "float64"),
                                             ("TQU", 6742, "float32"), ("IQU", 20224, "float64")])
def test_around_the_lds_limit(monkeypatch, form, streams, n, dtype):
    """One-sample baselines, as many as LDS holds and one more, against the plain form (same sums in another order).

    One iteration: with one-sample T baselines K is a multiple of a projector, so a second step divides by rounding.
    """
    from paper_1309_5609_amd import dst
    p = toy(n_samples=n, L=1, nside=4, streams=streams, mask_fraction=0.03)
    dp = dst.to_device(p, tod_dtype=dtype, psi_dtype=dtype)
    res = []
    for f in (form, 0):
        c = context(monkeypatch, f)
        res.append(dst.dst_solve(c, dp, tol=1e-30, max_iter=1))
        c.close()
    for k in ("baselines", "destriped_map", "binned_map"):
        # two operator applications of sums of up to n terms: n eps = 1e-11 each
        assert rel(res[0][k].cpu().numpy(), res[1][k].cpu().numpy()) < 1e-10, k


@pytest.mark.parametrize("form", [1, 2])
def test_group(monkeypatch, form):
    """An uneven batch whose problems all take the form."""
    from paper_1309_5609_amd import dst
    c = context(monkeypatch, form)
    probs = [toy(n_samples=30000, L=300, nside=16, cfg=330), toy(n_samples=6000, L=5, nside=4, cfg=331),
             toy(n_samples=12011, L=211, cfg=332, streams="T"), toy(n_samples=20000, L=400, cfg=333, streams="IQU"),
             toy(n_samples=20000, L=500, nside=16, cfg=334, streams="QU")]
    dps = [dst.to_device(p) for p in probs]
    _, out = dst.dst_solve_batched(c, dps, tol=1e-11, max_iter=2000)
    for p, dp, o in zip(probs, dps, out):
        one = dst.dst_solve(c, dp, tol=1e-11, max_iter=2000)
        assert abs(o["iterations"] - one["iterations"]) <= 1 + one["iterations"] // 50
        assert rel(o["baselines"].cpu().numpy(), one["baselines"].cpu().numpy()) < 1e-7
        assert rel(o["binned_map"].cpu().numpy(), one["binned_map"].cpu().numpy()) < 1e-12
    c.close()
