"""One-shot calls under stream capture: what the graph holds, and what calls before and after it may be.

Hits and validity are bit-exact; sums of h terms, each at most x, differ by at
most eps (h + 8) h x between two orders (the tolerance of the bucket form's
tests).
"""
import numpy as np
import pytest

from test_gpu_bucket import EPS, N_PIX, samples

pytestmark = pytest.mark.gpu


def problem(n, streams="TQU", weights=(1.0, 3.0, 3.0), n_pix=N_PIX, dtype=None):
    import torch
    from paper_1309_5609_amd import dst
    return dst.Problem(*samples(n, streams, dtype or torch.float64, "runs"), n_pix, 250, streams, weights)


def calls(name):
    from paper_1309_5609_amd import dst
    return {"bin": lambda c, p: dst.dst_bin(c, p)[0],
            "setup": lambda c, p: dst.dst_pixel_setup(c, p)[1],
            "reduce": lambda c, p: dst.dst_baseline_reduce(c, p, p.tod),
            "residual": lambda c, p: dst.dst_residual(c, p)}[name]


def capture(c, call, p):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = call(c, p)
    return g, out


def close(got, want, n):
    """Within the bound of sums of up to 3 n / N_PIX + 60 terms per pixel, or n / n_b per baseline, of values below 100."""
    h = max(3.0 * n / N_PIX + 60.0, 250.0)
    return bool(((got - want).abs() <= EPS * (h + 8.0) * h * 100.0).all())


# the captured call, and the calls on the same context after it: a longer timeline, larger records (data; block sums),
# a larger map
@pytest.mark.parametrize("name", ["bin", "setup", "reduce", "residual"])
def test_longer_calls_after_a_capture(name):
    import torch
    from paper_1309_5609_amd import dst
    c, e = dst.Context(0), dst.Context(0)
    p = problem(9_001)
    call = calls(name)
    call(c, p)
    torch.cuda.synchronize()
    g, got = capture(c, call, p)
    want = call(e, p)
    for later in (problem(3_000_001), problem(3_000_001, weights=(1.0, 3.0, 2.0)), problem(9_001, n_pix=2_000_000)):
        for other in ("setup", "bin", "residual"):
            calls(other)(c, later)
        torch.cuda.synchronize()
        # memory that the context gave back would be handed out again here
        torch.cuda.empty_cache()
        guard = [torch.full((k << 18,), 7, dtype=torch.int32, device="cuda") for k in (1, 4, 16, 64, 256)]
        got.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(bool((t == 7).all()) for t in guard)
        assert close(got, want, 9_001)
        del guard
    c.close()
    e.close()


EQ, NE = (1.0, 3.0, 3.0), (1.0, 3.0, 2.0)
WIDE = 3_200_000  # fits the buckets with equal q/u weights only


# the call before (eager), the captured one: every pair that needs no more than a map of as many pixels
@pytest.mark.parametrize("before,after", [
    (("bin", "T", EQ, 901, N_PIX), ("bin", "TQU", EQ, 901, N_PIX)),
    (("bin", "T", EQ, 901, N_PIX), ("bin", "TQU", NE, 901, N_PIX)),
    (("bin", "TQU", EQ, 901, N_PIX), ("bin", "QU", NE, 70_001, N_PIX)),
    (("bin", "T", EQ, 901, N_PIX), ("bin", "TQU", NE, 1_300_001, N_PIX)),      # several pieces
    (("setup", "T", EQ, 901, N_PIX), ("setup", "TQU", NE, 1_300_001, N_PIX)),
    (("setup", "TQU", EQ, 901, N_PIX), ("reduce", "TQU", NE, 901, N_PIX)),
    (("bin", "QU", EQ, 901, N_PIX), ("reduce", "TQU", EQ, 901, N_PIX)),
    (("residual", "T", EQ, 901, N_PIX), ("bin", "TQU", NE, 901, N_PIX)),
    (("residual", "QU", EQ, 901, N_PIX), ("residual", "QU", NE, 901, N_PIX)),
    (("bin", "TQU", EQ, 901, N_PIX), ("bin", "TQU", NE, 901, N_PIX // 9)),     # a smaller map
    (("bin", "T", EQ, 901, WIDE), ("bin", "TQU", NE, 901, WIDE)),              # buckets, then the atomic form
    (("residual", "TQU", EQ, 901, WIDE), ("residual", "TQU", NE, 901, WIDE)),
    (("bin", "TQU", EQ, 901, 7_000_000), ("bin", "TQU", NE, 901, N_PIX)),      # the atomic form, then a small map
])
def test_captured_call_is_accepted(before, after):
    import torch
    from paper_1309_5609_amd import dst
    c, e = dst.Context(0), dst.Context(0)
    name, streams, weights, n, n_pix = before
    calls(name)(c, problem(n, streams, weights, n_pix))
    torch.cuda.synchronize()
    name, streams, weights, n, n_pix = after
    p = problem(n, streams, weights, n_pix)
    if n_pix < N_PIX:
        p.pix %= n_pix
    g, got = capture(c, calls(name), p)
    for k in range(3):
        p.tod.mul_(-1.5)
        want = calls(name)(e, p)
        g.replay()
        torch.cuda.synchronize()
        assert close(got, want, n)
    c.close()
    e.close()
