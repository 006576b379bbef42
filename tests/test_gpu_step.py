"""PCG step length and stopping test finished inside the update and direction kernels, at the edges of their sizes.

Alone, a problem whose rescan leaves up to 4096 partials sums them in every
workgroup of the update; in a group, and beyond, one workgroup's kernel does.
The order of the sums is one and the same, so with equal launch shapes the bits
are equal.  The launch shapes chosen by size change the order of the sums only.
"""
import numpy as np
import pytest

from problems import toy

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


# 16 baselines per workgroup of the rescan with four per wavefront: 8, 64, 72, 1024, 1032, 4096 and 4104 partials
@pytest.mark.parametrize("n_b", [40, 1024, 1025, 16384, 16385, 65536, 65537])
@pytest.mark.parametrize("streams", ["T", "TQU"])
def test_step_alone_and_in_a_group(monkeypatch, streams, n_b):
    from paper_1309_5609_amd import dst
    p = toy(n_samples=3 * n_b - 1, L=3, nside=8, streams=streams, mask_fraction=0.02)
    other = toy(n_samples=701, L=7, nside=4, streams=streams)
    dp, do = dst.to_device(p), dst.to_device(other)
    run = dict(tol=1e-14, max_iter=6)
    by_size = dst.Context(0)
    free = dst.dst_solve(by_size, dp, **run)
    by_size.close()
    for k, v in {"DST_UNBIN_BPW": "4", "DST_BIN_LPP": "4", "DST_BIN_FORM": "0"}.items():
        monkeypatch.setenv(k, v)
    c = dst.Context(0)
    alone = dst.dst_solve(c, dp, **run)
    group = dst.dst_solve_batched(c, [dp, do], **run)[1][0]
    c.close()
    assert alone["iterations"] == group["iterations"] == free["iterations"]
    # (a group's closing binning, and so its map, has lanes of its own)
    assert np.array_equal(alone["baselines"].cpu().numpy(), group["baselines"].cpu().numpy())
    for k in ("baselines", "destriped_map"):
        a = alone[k].cpu().numpy()
        # six iterations of sums of up to 2e5 terms: below 1e-10
        assert rel(free[k].cpu().numpy(), a) < 1e-10, k
