"""Squared-L2 tables at the edges of their launch: plane counts on both sides of
each accumulator count (17, 33, 65 entries), more levels than one launch takes,
one-value levels, and values far below the level's largest (summed unscaled).
Tolerance as in test_gpu_l2.py: non-negative terms, each added with one
rounding, at most (n / 256 + 1100) 2^-53 relative for these sizes, below 1e-12."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _check(orc, xs, B):
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    dev = [torch.from_numpy(x).cuda() for x in xs]
    r = mdr.refactor(ctx, dev, B)
    r.l2_table(dev)
    for l, (x, lv) in enumerate(zip(xs, orc.refactor(xs, B))):
        np.testing.assert_allclose(np.array(r.l2(l)), orc.l2_table(x, lv), rtol=1e-12, atol=0, err_msg="level %d" % l)
    r.close()
    ctx.close()


@pytest.mark.parametrize("dtype,B", [(np.float32, 4), (np.float32, 16), (np.float32, 17), (np.float64, 16),
                                     (np.float64, 32), (np.float64, 33), (np.float64, 63)])
def test_plane_counts(orc, dtype, B):
    say("l2 planes", np.dtype(dtype).name, B)
    rng = np.random.default_rng(B)
    _check(orc, [rng.laplace(0, 1, n).astype(dtype) for n in (1, 0, 2047, 2049, 70_001)], B)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_more_levels_than_a_launch(orc, dtype):
    say("l2 levels", np.dtype(dtype).name)
    rng = np.random.default_rng(3)
    sizes = [int(n) for n in rng.integers(0, 300, 131)]
    sizes[63] = sizes[64] = sizes[130] = 0
    sizes[62] = 9001
    _check(orc, [rng.laplace(0, 2.0 ** (l % 7), n).astype(dtype) for l, n in enumerate(sizes)], 20)


def test_values_far_below_the_largest(orc):
    say("l2 tiny values")
    rng = np.random.default_rng(4)
    x = np.ldexp(rng.uniform(1, 2, 3000), rng.integers(-480, -420, 3000))  # 2^-400 below the largest and less
    x[1234] = 2.0 ** 40                                                    # its own residual is 0 from k = 1 on
    y = np.ldexp(rng.uniform(1, 2, 3000), rng.integers(-420, 41, 3000))
    _check(orc, [x, -x, y], 64)
