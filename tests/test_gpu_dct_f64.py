"""The FP64 DCT stages (even/odd split on the matrix cores, any side length) at
the sizes where they can go wrong: sides below a K step, odd sides (a middle
element without a mirror), remainders of a K step and of a tile in either
direction, and maps on both sides of the tile rule (32 x 32 below 224 tiles of
64 x 64, 64 x 64 from there on).  Reference: the same transform from dense
matrices in FP64.

Tolerance: the transform is orthonormal, so a stage's error is at most about
n u of its input's norm (n the side, u = 2^-53), and the two inverse stages
carry it through 1 / lambda_min = (n / pi)^2 at worst: |s - ref| <=
4 n u (n / pi)^2 ||r|| bounds it; the observed error is far below.  The
residual form L0 s = r - mean(r), free of that amplification, is checked to
16 n u ||r||_inf with the operator's norm 8 in place.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U64 = 2.0 ** -53
SIZES = [(1, 1), (1, 2), (2, 1), (1, 31), (3, 65), (31, 33), (32, 64), (63, 64), (65, 66), (96, 97),
         (127, 257), (200, 15), (509, 301), (896, 1023), (896, 1024), (1025, 961), (1000, 1101)]


def dct_matrix(n):
    k = torch.arange(n, device="cuda", dtype=torch.float64)
    c = torch.cos(math.pi * k[:, None] * (2 * k[None, :] + 1) / (2 * n)) * math.sqrt(2.0 / n)
    c[0] = math.sqrt(1.0 / n)
    return c


@pytest.mark.parametrize("M,N", SIZES)
def test_dct_f64(M, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    g = torch.Generator(device="cuda").manual_seed(M * 10000 + N)
    U = torch.rand(M, N, device="cuda", dtype=torch.float64, generator=g) + 0.1
    V = torch.rand(M, N, device="cuda", dtype=torch.float64, generator=g) + 0.1
    U[:, -1] = 0.0
    V[-1] = 0.0
    r = torch.randn(M, N, device="cuda", dtype=torch.float64, generator=g)
    with Context(0) as ctx:
        s = ctx.precond_apply(U, V, r, "dct", precision="fp64")
    if M * N == 1:
        assert float(s) == 0.0
        return
    A, B = dct_matrix(M), dct_matrix(N)
    km, kn = (torch.arange(n, device="cuda", dtype=torch.float64) for n in (M, N))
    lam = (2 - 2 * torch.cos(math.pi * km / M))[:, None] + (2 - 2 * torch.cos(math.pi * kn / N))
    lam[0, 0] = math.inf
    want = A.t().contiguous() @ ((A @ r @ B.t().contiguous()) / lam) @ B
    n = max(M, N)
    norm = float(r.norm())
    assert float((s - want).norm()) <= 4 * n * U64 * (n / math.pi) ** 2 * norm
    Ls = torch.zeros_like(s)
    dx, dy = s[:, 1:] - s[:, :-1], s[1:] - s[:-1]
    Ls[:, :-1] -= dx
    Ls[:, 1:] += dx
    Ls[:-1] -= dy
    Ls[1:] += dy
    scale = 8 * float(s.abs().max()) + float(r.abs().max())
    assert float((Ls - (r - r.mean())).abs().max()) <= 16 * n * U64 * scale


def test_dct_f64_batch_of_both_tiles_matches_single():
    """Maps of both tile sides in one launch: each map's result equals its
    single solve bit for bit (the tile side is the map's alone)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    rng = np.random.default_rng(4)
    psis = [torch.from_numpy(rng.uniform(-3.0, 3.0, s)).cuda()
            for s in ((70, 90), (1030, 900), (33, 200), (128, 128))]
    kw = dict(p=0.0, preconditioner="dct", precision="fp64", k_max=1, outer_tol=0.0, l_max=8)
    with Context(0) as ctx:
        phis, _, stats = ctx.batch(psis, **kw)
        for k, psi in enumerate(psis):
            one = ctx.solve(psi, **kw)
            assert stats[k]["inner_iters_total"] == one.stats["inner_iters_total"]
            assert torch.equal(phis[k], one.phi), psi.shape
