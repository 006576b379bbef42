"""Lists of the staged rescan in a problem group: none where one of a kind's problems is not dense enough to use them."""
import pytest

pytestmark = pytest.mark.gpu


def test_mixed_kind_holds_no_lists(monkeypatch):
    """A dense intensity problem (40 runs on each of 530,000 pixels) beside a short one, staging by size and off.

    The lists of the dense one would take 4 bytes a run and 40 KB for every 16 baselines, 100 MB.
    """
    import torch
    from paper_1309_5609_amd import dst
    n_pix = 530_000
    n = 40 * n_pix
    t = torch.arange(n, device="cuda")
    pix = ((t * 17) % n_pix).to(torch.int32)
    tod = torch.randn(1, n, device="cuda", dtype=torch.float32)
    ps = [dst.Problem(pix, None, tod, n_pix, 6000, "T", (1.0,) * 3),
          dst.Problem(pix[:50_000].clone(), None, tod[:, :50_000].contiguous(), n_pix, 500, "T", (1.0,) * 3)]

    def held(bpw):
        if bpw:
            monkeypatch.setenv("DST_UNBIN_BPW", bpw)
        else:
            monkeypatch.delenv("DST_UNBIN_BPW", raising=False)
        c = dst.Context(0)
        dst.dst_solve_batched(c, ps, max_iter=5)
        torch.cuda.synchronize()
        used = -torch.cuda.mem_get_info()[0]
        c.close()
        return used + torch.cuda.mem_get_info()[0]

    held("4")  # torch's own allocations are made
    plain, by_size, forced = held("4"), held(""), held("16")
    assert abs(by_size - plain) < 8 << 20, (plain, by_size)
    assert forced - plain > 80 << 20, (plain, forced)
