"""Short noise timelines (a last tile with few segments) against the head of a long one: the same bits.

A pair of segments is a function of the seed, the stream and its number alone,
whatever stands beside it in a tile, so a timeline cut short inside the second
segment of a pair keeps its values.  (Cut inside the first, that segment is
filtered with zeros beside it and rounds otherwise.)
"""
import pytest

pytestmark = pytest.mark.gpu


# one pair, two, about the end of a tile (4096 pairs of values), and a pair more
@pytest.mark.parametrize("segment", [4, 8, 64, 256, 1024, 2048, 4096])
@pytest.mark.parametrize("fknee", [0.0, 0.3])
def test_head_of_a_long_timeline(segment, fknee):
    import torch
    from paper_1309_5609_amd import dst
    c = dst.Context(0)
    args = (segment, 50.0, 1.5, fknee, 1.3)
    long = dst.dst_noise_generate(c, 11, 3, 40000, *args)
    for n in (segment + 1, 2 * segment - 1, 2 * segment, 3 * segment + 1, 8191, 8192, 8192 + segment + 1):
        assert -(-n // segment) % 2 == 0
        assert torch.equal(dst.dst_noise_generate(c, 11, 3, n, *args), long[:n]), n
        short = dst.dst_noise_generate(c, 11, 3, n, *args, dtype=torch.float32)
        assert torch.equal(short, long[:n].float()), n
    c.close()
