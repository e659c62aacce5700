"""Encoder workgroups of a mid-size pass against other launch shapes.

A pass of at most 4096 (f32) or 12288 (f64) tiles of 8192 values in the
register fast paths aims for one round of workgroups, a larger one for the
context's target.  On both sides of each limit, and at the smallest pass the
rule applies to, error tables, methods and stream sizes have to equal those of
a pass that walks more tiles a workgroup (tables and sizes are whole results:
no tolerance)."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _tables(mdr, ctx, x, B, target):
    ctx.set_launch(enc_target_wg=target, graphs=0)
    r = mdr.refactor(ctx, [x[:4099], x[4099:].clone()], B, mdr.default_params(group_planes=4))
    out = [(r.info(l)["E"], [r.stream(l, s)[1:] for s in range(-1, B)]) for l in range(2)]
    r.close()
    return out


@pytest.mark.parametrize("bits,tiles", [(32, 257), (32, 4095), (32, 4097), (64, 129), (64, 12287), (64, 12289)])
def test_rounds_do_not_change_results(bits, tiles):
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    n = tiles * 8192 - 4093  # with the small level: `tiles` tiles and one
    g = torch.Generator(device="cuda").manual_seed(tiles)
    x = torch.randn(n, device="cuda", generator=g, dtype=torch.float32 if bits == 32 else torch.float64)
    x *= torch.rand(n, device="cuda", generator=g, dtype=x.dtype) ** 6
    say("encoder rounds: bits", bits, "tiles", tiles, "values", n)
    assert _tables(mdr, ctx, x, bits, 2304) == _tables(mdr, ctx, x, bits, 300)
    ctx.close()
