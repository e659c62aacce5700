"""Placement of decoded units in memory: units of a power of two of bytes may not
make the reconstruction, which reads every plane's row at once, slower than units
a little smaller."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def test_power_of_two_units_are_not_slower():
    """17 decoded units of 8 MiB (2^24 f64 values), against units 1/262 smaller."""
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    us = {}
    for n in (1 << 24, (1 << 24) - 64 * 1001):
        x = [torch.full((n,), 0.7, dtype=torch.float64, device="cuda")]
        r = mdr.refactor(ctx, x, 64, mdr.default_params(group_planes=4, force_method=1))
        out = [torch.empty_like(x[0])]
        us[n] = 1e9
        for _ in range(20):
            ctx.set_timing(True)
            ctx.timing()
            rt = mdr.Retriever(ctx, r)
            rt.retrieve_planes([64], out)
            torch.cuda.synchronize()
            rt.close()
            us[n] = min(us[n], 1e3 * ctx.timing()["reconstruct"][0])
        ctx.set_timing(False)
        assert torch.equal(out[0], x[0])
        r.close()
        say("reconstruction of", n, "values:", us[n], "us")
    ctx.close()
    assert us[1 << 24] <= us[(1 << 24) - 64 * 1001]
