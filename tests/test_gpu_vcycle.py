"""One multigrid V-cycle, point by point, against a plain one in 64 bits.

A multigrid-preconditioned solve from zero that may do one iteration returns
x = alpha z with z = B r, r the right-hand side, B one V-cycle and alpha =
<r, z> / <z, A z>. The plain cycle is written with whole-grid shifts: red then
black half-sweep from zero, residual, full weighting (1/4, 1/2, 1/4 an axis),
the coarse correction by trilinear interpolation, black then red half-sweep;
the coarsest grid (at most 12 points a side, odd or below 8) is solved by
the DFT.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_20418_amd import inputs  # noqa: E402

pytestmark = pytest.mark.gpu


def six(x):
    return sum(torch.roll(x, s, d) for d in range(3) for s in (1, -1))


def vcycle(b, c=1.0):
    N = b.shape[0]
    if N % 2 or N // 2 < 4:
        k = 2.0 - 2.0 * torch.cos(2.0 * math.pi * torch.arange(N, dtype=b.dtype, device=b.device) / N)
        lam = c * (k[:, None, None] + k[None, :, None] + k[None, None, :])
        lam[0, 0, 0] = 1.0
        f = torch.fft.fftn(b) / lam
        f[0, 0, 0] = 0.0
        return torch.fft.ifftn(f).real
    i = torch.arange(N, device=b.device)
    red = (i[:, None, None] + i[None, :, None] + i[None, None, :]) % 2 == 0

    def sweep(x, where):
        return torch.where(where, (b / c + six(x)) / 6.0, x)
    x = sweep(sweep(torch.zeros_like(b), red), ~red)
    r = b - c * (6.0 * x - six(x))
    for d in range(3):
        r = 0.5 * r + 0.25 * (torch.roll(r, 1, d) + torch.roll(r, -1, d))
    e = vcycle(r[::2, ::2, ::2].contiguous(), c / 4.0)
    for d in range(3):
        e = torch.stack([e, 0.5 * (e + torch.roll(e, -1, d))], d + 1).flatten(d, d + 1)
    return sweep(sweep(x + e, ~red), red)


# one level (9); one workgroup for all (16, 24); ragged rows and chunks (18, 22, 36,
# 44); tiles of 8 rows (96, 112); rows in pieces, ragged and even (144, 176, 128);
# long chunks (192, 224)
@pytest.mark.parametrize("N", [9, 16, 18, 22, 24, 36, 44, 64, 96, 112, 128, 144, 176, 192, 224])
@pytest.mark.parametrize("precision", [0, 1])
def test_vcycle_point_by_point(N, precision):
    """FP64: the coarsest solve ends at 1e-14 of its right-hand side, times at
    most 45 (the condition of 12^3): 4.5e-13, and rounding. FP32 cycle: sums of
    up to 30 terms (2e-6) in four passes a level."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_20418_amd import maze

    def dev(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    print(f"case: V-cycle N {N} precision {precision}", flush=True)
    s = inputs.molten_nacl(max(2, N // 16), seed=N)
    x = maze.Session(dev(s.charges), dev(s.pos), s.box, s.box / N, tol=1e-300, max_iter=1,
                     precision=precision, flags=maze.MAZE_FLAG_MULTIGRID)
    out = x.solve(dev(s.pos + s.vel))
    assert out["stats"]["iters"] == 1
    q = x.grid(maze.GRID_Q)
    b = (4.0 * math.pi * N / s.box) * (q - q.mean())
    z = vcycle(b)
    az = 6.0 * z - six(z)
    want = (b * z).sum() / (z * az).sum() * z
    want = want - want.mean()
    levels, n = 1, N
    while n % 2 == 0 and n // 2 >= 4:
        levels, n = levels + 1, n // 2
    tol = 2e-12 if precision == 0 else 4 * 2e-6 * levels
    scale = want.abs().max().item()
    assert (out["field"] - want).abs().max().item() <= tol * scale
    x.close()
