"""Remainder passes of a batch's setup (one and two realizations keep narrower records) against the single solve."""
import numpy as np
import pytest

from test_gpu_batched import family, on_device

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


# passes of five realizations and the rest: 2; 3; 5 + 1; 5 + 2; 5 + 4; 5 + 5 + 1
@pytest.mark.parametrize("n_real", [2, 3, 6, 7, 9, 11])
@pytest.mark.parametrize("streams,dtype", [("T", "float64"), ("QU", "float64"), ("TQU", "float64"), ("TQU", "float32")])
def test_remainder(streams, dtype, n_real):
    from paper_1309_5609_amd import dst
    c = dst.Context(0)
    dps = on_device(family(n_real, streams=streams, mask_fraction=0.03), tod_dtype=dtype)
    _, res = dst.dst_solve_batched(c, dps, tol=1e-13, max_iter=3000)
    for d, out in zip(dps, res):
        one = dst.dst_solve(c, d, tol=1e-13, max_iter=3000)
        # both within 1e-9 of the solution, the binned map within 1e-12
        assert rel(out["baselines"].cpu().numpy(), one["baselines"].cpu().numpy()) < 2e-9
        assert rel(out["destriped_map"].cpu().numpy(), one["destriped_map"].cpu().numpy()) < 2e-9
        assert rel(out["binned_map"].cpu().numpy(), one["binned_map"].cpu().numpy()) < 2e-12
        assert np.array_equal(out["hits"].cpu().numpy(), one["hits"].cpu().numpy())
    c.close()
