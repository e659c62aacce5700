"""A field of more wavefronts than one grid dimension holds threads for: 15488 x
15488 rows of 129 f32 values (124 GB, and as much for the coefficients), 1.7 x 10^7
workgroups of 256 threads in the decomposition's one launch.  The values are
small whole numbers, so every mean and coefficient is exact and the field has to
come back as it was; coefficients are compared at the raw grid and on whole
planes of the finest level."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

N0 = N1 = 15488
N2 = 129


def test_grid_past_one_dimension():
    import torch

    import paper_2505_00227_amd as mdr
    torch.cuda.empty_cache()
    values = N0 * N1 * N2
    free, _ = torch.cuda.mem_get_info()
    if free < 8 * values + (6 << 30):
        pytest.skip(f"needs {8 * values >> 30} GiB of device memory, {free >> 30} free")
    say("multilevel grid:", values, "values,", free >> 30, "GiB free")
    u = torch.empty((N0, N1, N2), dtype=torch.float32, device="cuda")
    coeffs = torch.empty(values, dtype=torch.float32, device="cuda")
    base = torch.arange(N1 * N2, device="cuda", dtype=torch.int64).mul_(7919).remainder_(1021).view(N1, N2)

    def plane(i):
        return base.add(37 * i).remainder_(1021).to(torch.float32)

    for i in range(N0):
        u[i] = plane(i)
    steps = 2
    mdr.decompose(u, steps, coeffs)
    torch.cuda.synchronize()
    m = [(n + 3) // 4 for n in (N0, N1, N2)]
    raw = coeffs[:m[0] * m[1] * m[2]].view(m)
    for i in (0, 1, m[0] // 2, m[0] - 1):
        assert torch.equal(raw[i], plane(4 * i)[::4, ::4]), ("raw plane", i)
    # odd planes of the finest level lie whole and in row order: u - P, P between two even planes
    h = [(n + 1) // 2 for n in (N0, N1, N2)]
    first = h[0] * h[1] * h[2]
    for a in (1, N0 // 2 + 1, N0 - 1):
        at = first + a * N1 * N2 - (a + 1) // 2 * h[1] * h[2]
        got = coeffs[at:at + N1 * N2].view(N1, N2)
        p = [plane(a - 1), plane(a + 1)] if a + 1 < N0 else [plane(a - 1)]
        for q in p:  # along x, then y; the last odd node takes its left neighbour
            q[:, 1:-1:2] = (q[:, 0:-2:2] + q[:, 2::2]) * 0.5
            q[1:-1:2] = (q[0:-2:2] + q[2::2]) * 0.5
            q[-1] = q[-2]
        P = (p[0] + p[1]) * 0.5 if len(p) == 2 else p[0]
        assert torch.equal(got, plane(a) - P), ("coefficients of plane", a)
    u.zero_()
    mdr.recompose(coeffs, steps, u)
    torch.cuda.synchronize()
    wrong = torch.zeros((), dtype=torch.int64, device="cuda")
    for i in range(N0):
        wrong += (u[i] != plane(i)).sum()
    assert wrong.item() == 0
    del u, coeffs
    torch.cuda.empty_cache()
