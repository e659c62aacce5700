"""Recompositions of one step, which take their coarse nodes from level 0 itself:
lines, planes and volumes past what one workgroup's LDS holds, rows on both sides
of a wavefront's 256 nodes, packed short rows, every parity of the three sizes,
buffers that start at any value.  Bit for bit against the oracle; and a flat grid
may not take longer than 1.6 copies of it (1.3 as it is, 1.9 with a copy of level
0 into every second value of the field first)."""
import numpy as np
import pytest

from gpu_util import assert_same_bits, say
from oracle import multilevel as ml

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 8193), (1, 1, 20_000), (1, 1, 65_537), (1, 33, 257), (1, 34, 512), (1, 36, 513), (1, 9000, 1), (9001, 1, 1),
          (1, 3000, 3), (3000, 1, 4), (2, 70, 61), (3, 71, 62), (20, 21, 22), (21, 20, 23), (22, 22, 21), (9, 10, 255),
          (10, 9, 258), (5, 6, 1023)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("skip", [0, 1])
def test_one_step(dtype, skip):
    import torch

    import paper_2505_00227_amd as mdr
    rng = np.random.default_rng(skip)
    for shape in SHAPES:
        say("one step", np.dtype(dtype).name, shape, "start", skip)
        c = rng.standard_normal(int(np.prod(shape))).astype(dtype)
        c[::13] = -0.0
        want = ml.recompose(np.split(c, np.cumsum(ml.level_sizes(shape, 1))[:-1]), shape, 1)
        buf = torch.full((c.size + skip + 9,), float("nan"), dtype=torch.from_numpy(c).dtype, device="cuda")
        field = buf[skip:skip + c.size].view(shape)
        mdr.recompose(torch.from_numpy(np.concatenate([np.ones(skip, dtype), c])).cuda()[skip:], 1, field)
        assert_same_bits(field.cpu().numpy(), want, shape)
        assert torch.isnan(buf[:skip]).all() and torch.isnan(buf[skip + c.size:]).all()  # nothing beside it


def test_flat_grid_time():
    import torch

    import paper_2505_00227_amd as mdr
    shape = (1, 4000, 4000)
    c = torch.randn(16_000_000, dtype=torch.float64, device="cuda")
    u = torch.empty(shape, dtype=torch.float64, device="cuda")
    v = torch.empty_like(c)

    def us(f):
        best = 1e9
        for _ in range(30):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best

    copy, step = us(lambda: v.copy_(c)), us(lambda: mdr.recompose(c, 1, u))
    say("copy", copy, "us, one step", step, "us")
    assert step <= 1.6 * copy
