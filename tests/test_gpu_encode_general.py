"""The encoders of larger passes against the oracle, bit for bit.

Passes of more than 2^21 float32 or 2^20 float64 values walk tiles of 8192
values.  Here 64 workgroups take several such tiles each, from levels that start
on and off a 16-byte boundary and end inside a tile, so the state that a
workgroup carries from tile to tile counts: the general encoders (a group size
other than 4, or fewer planes than the type has) of both types, which the sizes
below those limits do not reach, and the register fast path of float32 (which
tests every value for its error keys: plane words are tested for them in the
fast path of float64 alone)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import assert_same_bits, compare_refactor, gpu_outputs, host, say, to_oracle_params

pytestmark = pytest.mark.gpu

TILE_VALUES = 8192
WORKGROUPS = 64


def _level(kind, n, dtype):
    rng = np.random.default_rng(n % 9973 + len(kind))
    if kind == "laplace":
        return rng.laplace(0, 1, n).astype(dtype)
    if kind == "ones":  # long runs of ones: every cut's maximum high
        return workloads.ones_runs_level(seed=n % 101, n=n, dtype=dtype)
    if kind == "constant":
        return workloads.piecewise_constant_level(seed=n % 103, n=n, dtype=dtype)
    if kind == "short":  # low planes empty: cuts without a bit below them
        return (rng.choice([-1.0, 1.0], n) * np.floor(rng.uniform(0, 1, n) * 512) / 512).astype(dtype)
    if kind == "late":  # the largest keys of every cut in the last values
        x = rng.uniform(-0.75, 0.75, n).astype(dtype)
        x[-3000:] = workloads.ones_runs_level(seed=3, n=3000, dtype=dtype)
        return x
    # wide: down to below every cut, zeros of both signs and subnormals among them
    bits = 24 if dtype == np.float32 else 53
    x = (rng.choice([-1.0, 1.0], n) * np.ldexp(rng.uniform(0.5, 1, n), -rng.integers(0, 40 + bits, n))).astype(dtype)
    x[::97] = 0.0
    x[1::97] = -0.0
    x[2::97] = np.finfo(dtype).smallest_subnormal
    return x


def _check(xs, skip, B, prm, ks):
    import torch

    import paper_2505_00227_amd as mdr
    values = sum(x.size for x in xs)
    assert values > (1 << 21 if xs[0].dtype == np.float32 else 1 << 20)
    tiles = sum(-(-x.size // TILE_VALUES) for x in xs)
    assert -(-tiles // WORKGROUPS) > 1
    say("general encoder:", xs[0].dtype, "values", values, "B", B, "m", prm.group_planes, "force", prm.force_method, "start", skip)
    ctx = mdr.Context(0)
    ctx.set_launch(enc_target_wg=WORKGROUPS, graphs=0)
    dev = [torch.from_numpy(np.concatenate([np.ones(skip, x.dtype), x])).cuda()[skip:] for x in xs]
    r = mdr.refactor(ctx, dev, B, prm)
    orc = oracle.refactor(xs, B, to_oracle_params(prm))
    compare_refactor(r, orc)
    rt = mdr.Retriever(ctx, r)
    outs = gpu_outputs(xs)
    for k in ks:
        rt.retrieve_planes([k] * len(xs), outs)
        for l, ol in enumerate(orc):
            assert_same_bits(host(outs[l]), ol.reconstruct(k), ("level", l, "k", k))
    rt.close()
    r.close()
    ctx.close()


@pytest.mark.parametrize("skip", [0, 1])
@pytest.mark.parametrize("kind", ["laplace", "ones", "constant", "short", "late", "wide"])
@pytest.mark.parametrize("B,m", [(40, 4), (64, 3)])
def test_general_f64(B, m, kind, skip):
    import paper_2505_00227_amd as mdr
    x = _level(kind, (1 << 20) + 70_001, np.float64)
    y = _level(kind, 5 * TILE_VALUES + 65, np.float64)
    _check([y, x], skip, B, mdr.default_params(group_planes=m), [m, B // m * m])


@pytest.mark.parametrize("skip", [0, 1])
@pytest.mark.parametrize("kind", ["laplace", "ones", "constant", "short", "late", "wide"])
@pytest.mark.parametrize("B,m", [(27, 4), (32, 3)])
def test_general_f32(B, m, kind, skip):
    import paper_2505_00227_amd as mdr
    x = _level(kind, (1 << 21) + 70_001, np.float32)
    y = _level(kind, 5 * TILE_VALUES + 33, np.float32)
    _check([y, x], skip, B, mdr.default_params(group_planes=m), [m, B // m * m])


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("B,m,force", [(0, 1, -1), (0, 8, 1), (5, 2, 2), (1, 1, -1), (0, 64, -1)])
def test_general_groups_and_methods(dtype, B, m, force):
    """Group sizes and plane counts at their ends, every method (B = 0: every plane)."""
    import paper_2505_00227_amd as mdr
    W = 32 if dtype == np.float32 else 64
    B = B or W
    m = min(m, B)
    n = (1 << (21 if dtype == np.float32 else 20)) + 12_345
    _check([_level("constant" if force == 1 else "wide", n, dtype)], 1, B,
           mdr.default_params(group_planes=m, force_method=force), [B // m * m])


@pytest.mark.parametrize("skip", [0, 1])
@pytest.mark.parametrize("kind", ["laplace", "ones", "constant", "short", "late", "wide"])
def test_fast_f32(kind, skip):
    import paper_2505_00227_amd as mdr
    x = _level(kind, 5 * WORKGROUPS * TILE_VALUES - 77 * skip, np.float32)
    _check([x], skip, 32, mdr.default_params(group_planes=4), [4, 32])


@pytest.mark.parametrize("bits,tiles", [(32, 257), (32, 4095), (32, 4097), (64, 129), (64, 12287), (64, 12289)])
def test_launch_shapes_give_equal_streams(bits, tiles):
    """The library's own workgroup count on both sides of its rule's limits, one
    asked for above it, and one with several times the tiles a workgroup: the
    whole serialized results are equal."""
    import torch

    import paper_2505_00227_amd as mdr
    n = tiles * TILE_VALUES - 4093  # with the small level: `tiles` tiles and one
    g = torch.Generator(device="cuda").manual_seed(tiles)
    x = torch.randn(n, device="cuda", generator=g, dtype=torch.float32 if bits == 32 else torch.float64)
    x *= torch.rand(n, device="cuda", generator=g, dtype=x.dtype) ** 6
    levels = [x[:4099], x[4099:].clone()]
    say("launch shapes: bits", bits, "tiles", tiles, "values", n)
    ctx = mdr.Context(0)
    blobs = []
    for target in (2304, 4608, 300):
        ctx.set_launch(enc_target_wg=target, graphs=0)
        r = mdr.refactor(ctx, levels, bits, mdr.default_params(group_planes=4))
        blobs.append(r.serialize())
        r.close()
        assert blobs[-1] == blobs[0], ("target", target)
    ctx.close()
