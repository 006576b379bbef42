"""dst_noise_generate over every split of the transform, against the noise oracle.

Segments of 2^2 .. 2^12 samples are filtered inside one tile, 2^13 .. 2^22 with
one column pass of radix 2 .. 1024, longer ones with two.  The bar is the noise
oracle's: 1e-12 of the RMS (the rounding of two FFTs of 2^23 points is about
1e-14 of it), 1e-6 for FP32 output.
"""
import numpy as np
import pytest

from oracle import noise as N

pytestmark = pytest.mark.gpu
RATE, SIGMA, FK, AL = 50.0, 1e-3, 0.05, 1.7


@pytest.fixture(scope="module")
def ctx():
    from paper_1309_5609_amd import dst
    c = dst.Context(0)
    yield c
    c.close()


def rms(x):
    return float(np.sqrt(np.mean(np.square(x))))


def segment(seed, stream, j, S):
    """Segment j of a timeline, by the oracle's own steps."""
    w = N.white_segment(seed, stream, j, S) * SIGMA
    return np.fft.irfft(np.fft.rfft(w) * N.filter_gain(S, RATE, FK, AL), n=S)


@pytest.mark.parametrize("m", range(2, 24))
def test_segment_lengths(ctx, m):
    """Segments of 2^m: three (an odd number, the last cut) up to 2^18, one beyond."""
    import torch
    from paper_1309_5609_amd import dst
    S = 1 << m
    n = 3 * S - S // 3 if m <= 18 else S - 5
    ref = np.concatenate([segment(m, 3, j, S) for j in range(-(-n // S))])[:n]
    got = dst.dst_noise_generate(ctx, m, 3, n, S, RATE, SIGMA, FK, AL)
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-12 * rms(ref)
    got = dst.dst_noise_generate(ctx, m, 3, n, S, RATE, SIGMA, FK, AL, dtype=torch.float32)
    assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-6 * max(rms(ref), float(np.max(np.abs(ref))))


@pytest.mark.parametrize("m", [4, 13])
def test_past_the_buffer(ctx, m):
    """More segment pairs than the buffer (2^25 complex values) or a first wave of tiles holds."""
    from paper_1309_5609_amd import dst
    S = 1 << m
    last = (1 << 26) // S  # index of the last segment, alone in its pair
    n = last * S + S // 2 + 1
    got = dst.dst_noise_generate(ctx, 5, 2, n, S, RATE, SIGMA, FK, AL)
    for j in (0, last // 2, last - 1, last):
        ref = segment(5, 2, j, S)[:n - j * S]
        assert np.max(np.abs(got[j * S:(j + 1) * S].cpu().numpy() - ref)) <= 1e-12 * max(rms(ref), SIGMA)
