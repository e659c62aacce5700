"""Retrieval of constant and nearly constant levels, whose planes are streams of
one-bit codes: decode tables at every limit on the code length against the
oracle, for several lane counts."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_same_bits, compare_refactor, gpu_outputs, host, say, to_oracle_params, upload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("lmax", [8, 9, 10, 11, 12])
def test_tables_of_short_codes(dtype, lmax):
    import paper_2505_00227_amd as mdr
    rng = np.random.default_rng(lmax)
    W = 32 if dtype == np.float32 else 64
    n = 70_001
    rare = np.full(n, 0.7, dtype)
    rare[rng.integers(0, n, 40)] = rng.uniform(0.1, 0.6, 40)
    xs = [np.zeros(n, dtype), np.full(n, 0.7, dtype), rare,
          (np.ldexp(rng.uniform(0.5, 1, n), -rng.geometric(0.5, n)) * rng.choice([-1, 1], n)).astype(dtype)]
    say("tables:", np.dtype(dtype).name, "lmax", lmax)
    ctx = mdr.Context(0)
    prm = mdr.default_params(group_planes=4, huf_lmax=lmax, force_method=2)
    r = mdr.refactor(ctx, upload(xs), W, prm)
    orc = oracle.refactor(xs, W, to_oracle_params(prm))
    compare_refactor(r, orc)
    outs = gpu_outputs(xs)
    for lanes in (0, 1, 4, 16, 64):
        ctx.set_decode_lanes(lanes)
        rt = mdr.Retriever(ctx, r)
        for k in (4, W):
            rt.retrieve_planes([k] * len(xs), outs)
            for l, ol in enumerate(orc):
                assert_same_bits(host(outs[l]), ol.reconstruct(k), ("lanes", lanes, "level", l, "k", k))
        rt.close()
    r.close()
    ctx.close()
