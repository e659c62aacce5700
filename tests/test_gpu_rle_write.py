"""Run-length streams of units with long constant stretches.

The writer looks from a tile (4096 words) that starts a run for the next tile
that starts one, 256 tiles a step.  Streams are compared with the oracle's for
gaps of none, some and more than 256 tiles with the starts at the tiles' edges;
and the writing of units with hardly any run may not take longer than that of
units with a run start in every tile, whose search ends at the next tile."""
import numpy as np
import pytest

import oracle
from gpu_util import compare_refactor, say, to_oracle_params, upload

pytestmark = pytest.mark.gpu

TILE = 4096  # words of a run-length tile


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("at", [(), (0,), (TILE - 1,), (TILE,), (2 * TILE + 7, 5 * TILE - 1), (39_999,), (1, 2, 30_000, 39_998)])
def test_gaps_against_the_oracle(dtype, at):
    """One unit of every plane, 40000 words a plane (312 tiles in 32 planes), zero but for single values."""
    import paper_2505_00227_amd as mdr
    W = 32 if dtype == np.float32 else 64
    x = np.zeros(40_000 * W, dtype)
    for k, w in enumerate(at):  # one value in the word
        x[w * W + (7 * k) % W] = [0.75, -0.3, 1.0, 0.6][k]
    say("run-length gaps:", np.dtype(dtype).name, at)
    ctx = mdr.Context(0)
    prm = mdr.default_params(group_planes=W, force_method=1)
    r = mdr.refactor(ctx, upload([x]), W, prm)
    compare_refactor(r, oracle.refactor([x], W, to_oracle_params(prm)))
    r.close()
    ctx.close()


def test_constant_units_are_not_slower():
    """2^28 values in one unit of 32 planes (65536 tiles): zeros, against values that alternate from tile to tile."""
    import torch

    import paper_2505_00227_amd as mdr
    n = 1 << 28
    ctx = mdr.Context(0)
    prm = mdr.default_params(group_planes=32, force_method=1)
    ms = {}
    for name in ("alternating", "zeros"):
        x = torch.zeros(n, dtype=torch.float32, device="cuda")
        if name == "alternating":
            x.view(-1, 2, TILE * 32)[:, 1] = 1 - 2.0 ** -24
        best = 1e9
        for _ in range(4):
            ctx.set_timing(True)
            ctx.timing()
            mdr.refactor(ctx, [x], 32, prm).close()
            best = min(best, ctx.timing()["lossless"][0])
        ctx.set_timing(False)
        ms[name] = best
        say("run-length pass:", name, "lossless stage", best, "ms")
    ctx.close()
    assert ms["zeros"] <= ms["alternating"]
