"""The encoder of small passes against the oracle, bit for bit: sizes at the edges
of its lanes (4 values), blocks (32), tiles (1024 values) and workgroup ranges,
levels that start at any alignment, both types, plane counts and groups of every
kind, and special values; and a pass of one value more than it takes."""
import numpy as np
import pytest

import workloads
from gpu_util import compare_refactor, say, to_oracle_params

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 4, 5, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 2047, 2081, 4096 + 37, 33 * 1024 + 1]


def _check(orc, xs, B, prm, offset=0, wg=0):
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    if wg:
        ctx.set_launch(enc_target_wg=wg)
    dev = []
    for x in xs:  # levels back to back in one buffer start at any value
        buf = torch.zeros(x.size + offset + 4, dtype=torch.from_numpy(x).dtype, device="cuda")
        buf[offset:offset + x.size] = torch.from_numpy(x).cuda()
        dev.append(buf[offset:offset + x.size])
    r = mdr.refactor(ctx, dev, B, prm)
    compare_refactor(r, orc.refactor(xs, B, to_oracle_params(prm)))
    r.close()
    ctx.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("frac,m", [(1.0, 4), (1.0, 1), (0.7, 3), (0.03, 1), (0.5, 64)])
def test_sizes(orc, dtype, frac, m):
    import paper_2505_00227_amd as mdr
    W = 32 if dtype == np.float32 else 64
    B = max(1, int(W * frac))
    say("small encoder", np.dtype(dtype).name, B, m)
    rng = np.random.default_rng(B + m)
    prm = mdr.default_params(group_planes=min(m, B), t_s_bytes=64)
    _check(orc, [rng.laplace(0, 2.0 ** (i % 5 - 2), n).astype(dtype) for i, n in enumerate(SIZES)], B, prm, offset=m % 4)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("wg", [64, 65536])
def test_ranges_and_special_values(orc, dtype, wg):
    import paper_2505_00227_amd as mdr
    say("small encoder values", np.dtype(dtype).name, wg)
    rng = np.random.default_rng(wg)
    W = 32 if dtype == np.float32 else 64
    fi = np.finfo(dtype)
    sp = np.array([0.0, -0.0, fi.tiny, -fi.tiny, fi.smallest_subnormal, -fi.smallest_subnormal, 1.0, -1.0, 1 - fi.epsneg],
                  dtype)
    xs = [workloads.ones_runs_level(5, 150_000, dtype), workloads.piecewise_constant_level(6, 130_001, dtype),
          np.zeros(3000, dtype), np.resize(sp, 2500), np.array([fi.max, -fi.max, fi.tiny], dtype), np.empty(0, dtype),
          rng.laplace(0, 1, 200_000).astype(dtype)]
    _check(orc, xs, W, mdr.default_params(group_planes=4, t_cr_milli=1000), wg=wg)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_the_limit(orc, dtype, over):
    import paper_2505_00227_amd as mdr
    n = (1 << (21 if dtype == np.float32 else 20)) + over
    say("small encoder limit", np.dtype(dtype).name, n)
    x = np.random.default_rng(n).laplace(0, 1, n).astype(dtype)
    _check(orc, [x], 32 if dtype == np.float32 else 64, mdr.default_params(group_planes=4))
