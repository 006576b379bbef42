"""Solves of one and of several components in turn on one context: each expects the other's form of the step."""
import numpy as np
import pytest

from problems import toy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 4])  # with the captured graph and without
def test_components_in_turn(flags):
    import torch
    from paper_1309_5609_amd import dst

    def problem(parts, streams):
        p = toy(n_samples=20000, L=250, nside=16, streams=streams)
        p.pix[:] = p.pix + p.n_pix * ((np.arange(len(p.pix)) // 250) % parts)
        dp = dst.to_device(p)
        dp.n_pix = parts * p.n_pix
        return dp

    ps = [problem(parts, streams) for parts, streams in ((1, "TQU"), (2, "TQU"), (3, "T"), (1, "T"), (2, "TQU"), (1, "QU"))]
    c = dst.Context(0)
    for p in ps + ps[::-1]:
        out = dst.dst_solve(c, p, tol=1e-12, max_iter=1000, flags=flags)
        fresh = dst.Context(0)
        want = dst.dst_solve(fresh, p, tol=1e-12, max_iter=1000, flags=flags)
        fresh.close()
        assert out["iterations"] == want["iterations"] and out["n_components"] == want["n_components"]
        assert torch.equal(out["baselines"], want["baselines"])
        assert torch.equal(out["destriped_map"], want["destriped_map"])
    c.close()
