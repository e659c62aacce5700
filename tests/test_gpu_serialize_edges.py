"""Serialization with the payloads' CRC-32 computed on the device: payload sizes
at the edges of its blocks (4096 words) and of the staging buffer (256 KiB), and
payloads of every method together, byte for byte against the oracle's blob (whose
CRC is pinned to zlib's); a blob loads back to equal bytes, and a flipped bit in
any payload is found."""
import numpy as np
import pytest

import oracle
from gpu_util import say, to_oracle_params

pytestmark = pytest.mark.gpu


def _round_trip(orc, xs, B, prm, flips):
    import torch

    import paper_2505_00227_amd as mdr
    ctx = mdr.Context(0)
    r = mdr.refactor(ctx, [torch.from_numpy(x).cuda() for x in xs], B, prm)
    blob = r.serialize()
    op = to_oracle_params(prm)
    assert blob == oracle.serialize(orc.refactor(xs, B, op), op)
    assert mdr.Refactored.deserialize(ctx, blob).serialize() == blob
    for at in flips(blob, r):
        bad = bytearray(blob)
        bad[at] ^= 0x10
        with pytest.raises(mdr.MdrError) as ei:
            mdr.Refactored.deserialize(ctx, bytes(bad))
        assert ei.value.status == mdr.MDR_ERR_CORRUPT_STREAM, at
    r.close()
    ctx.close()


@pytest.mark.parametrize("words", [1, 2, 255, 257, 4095, 4096, 4097, 8192, 65535, 65536, 65537])
def test_payload_sizes(orc, words):
    import paper_2505_00227_amd as mdr
    say("serialize", words)
    rng = np.random.default_rng(words)
    xs = [rng.laplace(0, 1, 32 * words).astype(np.float32), rng.laplace(0, 1, 40).astype(np.float32)]
    prm = mdr.default_params(group_planes=2, force_method=0)
    _round_trip(orc, xs, 5, prm, lambda blob, r: (len(blob) - 9, 56 + 40 + 8 * 6 + 16 * 6 + 8 + 4 * (words // 2)))


@pytest.mark.parametrize("force", [-1, 1, 2])
def test_methods_together(orc, force):
    import paper_2505_00227_amd as mdr
    import workloads
    say("serialize methods", force)
    rng = np.random.default_rng(9)
    xs = [workloads.piecewise_constant_level(3, 90001, np.float64), np.zeros(5000), np.empty(0),
          rng.laplace(0, 1, 30011)]
    prm = mdr.default_params(group_planes=4, force_method=force, t_cr_milli=1000)
    _round_trip(orc, xs, 64, prm, lambda blob, r: rng.integers(len(blob) - 100000, len(blob) - 64, 6))
