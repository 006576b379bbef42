"""Outputs beside an error: after a breakdown they hold the last iterate."""
import ctypes

import numpy as np
import pytest

from problems import toy

pytestmark = pytest.mark.gpu


# workgroups of the residual update: 1, 40 and 282; the last two of several components (a kernel of its own for the step)
@pytest.mark.parametrize("streams,n_b,parts", [("T", 40, 1), ("TQU", 3400, 1), ("TQU", 24000, 1), ("T", 400, 2),
                                               ("TQU", 3400, 3)])
def test_breakdown_returns_the_last_iterate(streams, n_b, parts):
    """A tolerance that is never met: past convergence p loses all but the null space and p.Kp falls to 0 or below.

    The outputs have the bits of a solve that is stopped at that iteration.
    """
    import torch
    from paper_1309_5609_amd import dst
    p = toy(n_samples=6 * n_b, L=6, nside=8, streams=streams)
    p.pix[:] = p.pix + p.n_pix * ((np.arange(len(p.pix)) // 6) % parts)
    dp = dst.to_device(p)
    dp.n_pix = parts * p.n_pix
    c = dst.Context(0)

    def run(max_iter):
        a = torch.zeros((dp.n_streams, dp.n_baselines), dtype=torch.float64, device="cuda")
        m = torch.zeros((dp.n_pix, 3), dtype=torch.float64, device="cuda")
        s, opts, info = dp.c_struct(0, need_tod=True), dst.dst_solve_opts(), dst.dst_solve_info()
        opts.tol, opts.max_iter = 5e-324, max_iter
        rc = c.lib.dst_solve(c.handle, ctypes.byref(s), ctypes.byref(opts), dst._ptr(a), dst._ptr(m), None, None,
                             ctypes.byref(info), dst._stream())
        return dst.STATUS[rc], info.iterations, a, m

    status, n, a, m = run(200000)
    assert status == "DST_EBREAKDOWN" and 10 < n < 200000
    status, n2, a2, m2 = run(n)
    assert status == "DST_ENOCONV" and n2 == n
    assert torch.equal(a, a2) and torch.equal(m, m2)
    c.close()
