"""Huffman code construction in the selection kernel at its edges: one, two and
256 present symbols, equal counts (every merge a tie), counts that make the
tree as deep as they can, and every limit on the code length, compared with the
oracle's streams byte for byte.  Inputs are sixteen-bit patterns written as
exact float32 values, so that the byte counts of the plane groups are chosen."""
import numpy as np
import pytest

from gpu_util import compare_refactor, say, to_oracle_params

pytestmark = pytest.mark.gpu


def _bytes_for(kind, n, rng):
    if kind == "one":
        return np.full(n, 0x5A, np.uint8)
    if kind == "two":
        return np.where(rng.random(n) < 0.1, 0x5A, 0x00).astype(np.uint8)
    if kind == "equal":  # 256 symbols, the same count each
        return np.resize(np.arange(256, dtype=np.uint8), n)
    if kind == "fibonacci":  # the deepest tree the size allows
        f = [1, 1]
        while sum(f) + f[-1] + f[-2] < n:
            f.append(f[-1] + f[-2])
        b = np.repeat(np.arange(len(f), dtype=np.uint8), f)
        return np.concatenate([b, np.full(n - b.size, len(f) - 1, np.uint8)])
    p = 0.5 ** (np.arange(256) / {"steep": 1.0, "skewed": 6.0, "flat": 60.0}[kind])
    return rng.choice(256, n, p=p / p.sum()).astype(np.uint8)


def _values(b):
    """float32 values whose planes of weight 2^0 and 2^-1 .. hold the bytes: 8
    bytes become 64 bits, one bit a value, in the second-highest plane."""
    bits = np.unpackbits(b, bitorder="little").astype(np.float32)
    return (1.0 + bits * 0.5).astype(np.float32)


@pytest.mark.parametrize("threads", [256, 512, 1024])
@pytest.mark.parametrize("kind", ["one", "two", "equal", "fibonacci", "steep", "skewed", "flat"])
def test_codes_match_oracle(orc, kind, threads):
    import torch

    import paper_2505_00227_amd as mdr
    say("select", kind, threads)
    rng = np.random.default_rng(sum(map(ord, kind)))
    xs = [_values(_bytes_for(kind, n, rng)) for n in (8192, 40000)]
    xs.append(rng.laplace(0, 1, 70000).astype(np.float32))
    ctx = mdr.Context(0)
    ctx.set_select_threads(threads)
    dev = [torch.from_numpy(x).cuda() for x in xs]
    for m, lmax, t_cr, force in ((1, 12, 1000, -1), (4, 8, 2000, -1), (2, 12, 2000, 2), (1, 9, 1000, 2), (4, 12, 7000, -1)):
        prm = mdr.default_params(group_planes=m, huf_lmax=lmax, t_cr_milli=t_cr, force_method=force)
        r = mdr.refactor(ctx, dev, 32, prm)
        compare_refactor(r, orc.refactor(xs, 32, to_oracle_params(prm)))
        r.close()
    ctx.close()
