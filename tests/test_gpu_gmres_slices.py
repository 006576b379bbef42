"""GMRES orthogonalisation at the edges of its slices (256 values, at most 256 slices) and of the vectors taken together."""
import numpy as np
import pytest

from problems import toy

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


# values of the basis vectors: below, at and past one slice, a remainder wave, and past 256 slices; eight vectors at a time
@pytest.mark.parametrize("streams,n_b", [("T", 63), ("T", 256), ("T", 257), ("QU", 128), ("TQU", 107), ("T", 65537)])
@pytest.mark.parametrize("restart", [7, 8, 9, 126])
def test_gmres_against_cg(streams, n_b, restart):
    from paper_1309_5609_amd import dst
    p = toy(n_samples=40 * n_b - 3, L=40, nside=8, streams=streams)
    c = dst.Context(0)
    dp = dst.to_device(p)
    cg = dst.dst_solve(c, dp, tol=1e-13, max_iter=3000)
    gm = dst.dst_solve(c, dp, tol=1e-13, max_iter=3000, flags=dst.DST_SOLVE_GMRES, restart=restart)
    assert gm["converged"] and gm["true_rel_residual"] < 1e-11
    for k in ("baselines", "destriped_map"):
        # both within 1e-9 of the solution, as against the oracle
        assert rel(gm[k].cpu().numpy(), cg[k].cpu().numpy()) < 2e-9, k
    c.close()
