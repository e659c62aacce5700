"""Error keys found from plane words, against the oracle.

From a workgroup's second tile on, the encoder of 32 float32 (64 float64)
planes in groups of 4 tests plane words for runs of ones below each cut and
looks only at the values a run flags; cuts whose running maximum is low are
taken directly, and with many of those the per-value test runs instead.  These
levels give every workgroup several tiles and drive each of those branches:
wide and narrow exponent ranges, significands that leave the low planes empty
(per-value test), all-ones significands (every value flagged), keys that rise
in the last tiles, values below every cut, zeros, subnormals, and a start that
is not 16-byte aligned with a ragged end.  Every table, method and stream has
to equal the oracle's exactly."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import compare_refactor, say, to_oracle_params

pytestmark = pytest.mark.gpu


def _level(kind, n, dtype):
    rng = np.random.default_rng(n + len(kind))
    bits = 24 if dtype == np.float32 else 53
    sign = rng.choice([-1.0, 1.0], n)
    if kind == "uniform":
        x = rng.uniform(-1, 1, n)
    elif kind == "wide":  # down to below every cut
        x = sign * np.ldexp(rng.uniform(0.5, 1, n), -rng.integers(0, 30 + bits, n))
    elif kind == "short":  # low planes empty
        x = sign * np.floor(rng.uniform(0, 1, n) * 1024) / 1024
    elif kind == "ones":  # every significand all ones
        x = sign * np.ldexp(1 - 2.0 ** -bits, -rng.integers(0, 8, n))
    elif kind == "late":  # the largest keys of every cut in the last values
        x = rng.uniform(-1, 1, n) * 0.75
        x[-4096:] = workloads.ones_runs_level(seed=5, n=4096, dtype=dtype)
    elif kind == "sparse":
        x = np.where(rng.uniform(0, 1, n) < 0.9, -0.0, rng.standard_normal(n))
    else:  # subnormal: the lowest cuts lie below the smallest value of the type
        x = np.ldexp(rng.uniform(-1, 1, n), -120 if dtype == np.float32 else -1012)
    return x.astype(dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["uniform", "wide", "short", "ones", "late", "sparse", "subnormal"])
def test_keys_by_plane(kind, dtype):
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    ctx.set_launch(enc_target_wg=64, graphs=0)
    B = 32 if dtype == np.float32 else 64
    prm = mdr.default_params(group_planes=4)
    op = to_oracle_params(prm)
    for n, skip in ((4 * 64 * 8192, 0), (2_200_000 + 7, 1)):
        x = _level(kind, n + skip, dtype)
        say("keys by plane:", kind, dtype.__name__, "values", n, "start", skip)
        r = mdr.refactor(ctx, [torch.from_numpy(x).cuda()[skip:]], B, prm)
        compare_refactor(r, oracle.refactor([x[skip:]], B, op))
        r.close()
    ctx.close()
