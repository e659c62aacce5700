"""Lossless plan at its unit-count limit, against the oracle.

A pass of at most 1024 units plans its Huffman chunks and run-length tiles in
every workgroup of the counting launch, a larger one in a launch of its own.
Batches on both sides of the limit, and one unit, coded by each forced method
and by the selection's own choice, have to give the oracle's streams."""
import numpy as np
import pytest

import oracle
from gpu_util import say, to_oracle_params, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("force", [-1, 1, 2])
@pytest.mark.parametrize("nvars", [1, 255, 256, 257])  # four units a variable
def test_units_at_the_limit(nvars, force):
    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    rng = np.random.default_rng(nvars)
    vs = [[(rng.standard_normal(int(n)) * (rng.uniform(0, 1, int(n)) < 0.2)).astype(np.float32)]
          for n in rng.integers(1, 3000, nvars)]
    p = mdr.default_params(group_planes=1, t_s_bytes=0, force_method=force)
    op = to_oracle_params(p)
    say("units:", 4 * nvars, "force", force)
    rs = mdr.refactor_batch(ctx, [upload(v) for v in vs], 3, p)
    for i, (r, v) in enumerate(zip(rs, vs)):
        assert r.serialize() == oracle.serialize(oracle.refactor(v, 3, op), op), ("variable", i, v[0].size)
    del rs
    ctx.close()
