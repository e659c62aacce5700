"""Multilevel decomposition and recomposition at the edges of their launches: rows
on both sides of a wavefront's 256 nodes and of the 252 that the fused last two
steps of a recomposition take, short rows packed into a wavefront, single rows
and planes, grids on both sides of what the first steps' workgroup holds, and
step counts that leave each kernel alone.  Bit for bit against the oracle."""
import numpy as np
import pytest

from gpu_util import assert_same_bits, say
from oracle import multilevel as ml

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (1, 1, 5), (1, 6, 4), (66, 1, 3), (3, 130, 9), (2, 2, 255), (3, 2, 257), (2, 5, 253), (1, 4, 505),
          (5, 1, 1021), (17, 33, 64), (9, 129, 65), (33, 37, 251), (31, 34, 252), (32, 35, 253), (33, 33, 258),
          (40, 17, 505), (3, 3, 4099), (129, 130, 17), (70, 71, 3)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("nsteps", [0, 1, 2, 3, 6])
def test_edges(dtype, nsteps):
    import torch

    import paper_2505_00227_amd as mdr
    rng = np.random.default_rng(nsteps)
    for shape in SHAPES:
        say("multilevel edges", np.dtype(dtype).name, nsteps, shape)
        u = rng.standard_normal(shape).astype(dtype)
        coeffs = torch.full((u.size,), float("nan"), dtype=torch.from_numpy(u).dtype, device="cuda")
        mdr.decompose(torch.from_numpy(u).cuda(), nsteps, coeffs)
        assert_same_bits(coeffs.cpu().numpy(), ml.concat(ml.decompose(u, nsteps)), ("decompose", shape))
        c = rng.standard_normal(u.size).astype(dtype)
        want = ml.recompose(np.split(c, np.cumsum(ml.level_sizes(shape, nsteps))[:-1]), shape, nsteps)
        # two starts of the output: no value of it is read before it is written
        for fill in (float("nan"), 3.0):
            field = torch.full(shape, fill, dtype=coeffs.dtype, device="cuda")
            mdr.recompose(torch.from_numpy(c).cuda(), nsteps, field)
            assert_same_bits(field.cpu().numpy(), want, ("recompose", shape, fill))
