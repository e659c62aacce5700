"""The G-lane Huffman decoder on both sides of the chunk count from which its
workgroups take 64 chunks instead of 16, with remainders of either, against the
one-thread decoder (itself pinned to the oracle) bit for bit: streams of one-bit
codes, of skewed and of flat ones, at every limit on the code length."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lmax", [8, 12])
@pytest.mark.parametrize("chunks", [15, 17, 1000, 8191, 16383, 16384, 16399])
def test_lane_counts_agree(chunks, lmax):
    import torch

    import paper_2505_00227_amd as mdr
    say("wide decode", chunks, lmax)
    g = torch.Generator("cuda").manual_seed(chunks)
    n = chunks * 2048  # a plane is `chunks` chunks of 256 bytes; k planes and the signs decode k + 1 of them
    u = torch.rand(n, device="cuda", generator=g)
    # planes 0 .. 2: nearly always zero (runs of one-bit codes), skewed, flat
    x = (u < 1e-4).float() * 0.5 + (torch.rand(n, device="cuda", generator=g) < 0.1).float() * 0.25 \
        + (torch.rand(n, device="cuda", generator=g) < 0.5).float() * 0.125
    x[0] = 0.5
    ctx = mdr.Context(0)
    r = mdr.refactor(ctx, [x], 3, mdr.default_params(group_planes=1, t_s_bytes=0, force_method=2, huf_lmax=lmax))
    for k in (1, 2, 3):
        got = []
        for lanes in (1, 0, 16):
            ctx.set_decode_lanes(lanes)
            out = [torch.empty_like(x)]
            mdr.Retriever(ctx, r).retrieve_planes([k], out)
            got.append(out[0].view(torch.int32))
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2]), k
    assert torch.equal(got[0], x.view(torch.int32))  # every bit of these values is in three planes
    r.close()
    ctx.close()
