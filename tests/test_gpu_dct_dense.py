"""The dense MFMA DCT stages (mixed path, sides that are not all multiples of
128) where they can go wrong: sides around a K step of 64 and its half,
remainders of a tile in either direction, odd sides (unaligned rows), maps on
both sides of the tile rule (32 x 32 below 192 tiles of 64 x 64).  Reference:
dense transforms in FP64; tolerances those of the other DCT applies, relative
to max |s| (split bf16 2e-4, scaled fp16 1e-2).
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 2), (2, 1), (3, 40), (31, 65), (32, 96), (64, 97), (63, 129), (200, 33), (250, 191),
         (768, 1000), (833, 959), (900, 1025)]


def dct_matrix(n):
    k = torch.arange(n, device="cuda", dtype=torch.float64)
    c = torch.cos(math.pi * k[:, None] * (2 * k[None, :] + 1) / (2 * n)) * math.sqrt(2.0 / n)
    c[0] = math.sqrt(1.0 / n)
    return c


@pytest.mark.parametrize("mode,rel", [("split_bf16", 2e-4), ("fp16_scaled", 1e-2)])
@pytest.mark.parametrize("M,N", SIZES)
def test_dct_dense(mode, rel, M, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    g = torch.Generator(device="cuda").manual_seed(M * 10000 + N)
    U = torch.rand(M, N, device="cuda", generator=g) + 0.1
    V = torch.rand(M, N, device="cuda", generator=g) + 0.1
    U[:, -1] = 0.0
    V[-1] = 0.0
    r = torch.randn(M, N, device="cuda", generator=g)
    with Context(0) as ctx:
        s = ctx.precond_apply(U, V, r, "dct", precision="mixed", dct_mode=mode).double()
    A, B = dct_matrix(M), dct_matrix(N)
    km, kn = (torch.arange(n, device="cuda", dtype=torch.float64) for n in (M, N))
    lam = (2 - 2 * torch.cos(math.pi * km / M))[:, None] + (2 - 2 * torch.cos(math.pi * kn / N))
    lam[0, 0] = math.inf
    want = A.t().contiguous() @ ((A @ r.double() @ B.t().contiguous()) / lam) @ B
    assert float((s - want).abs().max()) <= rel * float(want.abs().max())


@pytest.mark.parametrize("mode", ["split_bf16", "fp16_scaled"])
def test_dct_dense_batch_of_both_tiles_matches_single(mode):
    """Maps of both tile sides in one launch: each map's result equals its
    single solve bit for bit (the tile side is the map's alone).  The 128 x 128
    map is along for the launch only: by itself it takes the even/odd kernels,
    whose arithmetic differs."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    rng = np.random.default_rng(6)
    psis = [torch.from_numpy(rng.uniform(-3.0, 3.0, s)).cuda()
            for s in ((70, 90), (1030, 900), (33, 200), (128, 128), (801, 1000))]
    kw = dict(p=0.0, preconditioner="dct", precision="mixed", dct_mode=mode, k_max=1, outer_tol=0.0)
    with Context(0) as ctx:
        phis, _, stats = ctx.batch(psis, **kw)
        for k, psi in enumerate(psis):
            if psi.shape[0] % 128 == 0 and psi.shape[1] % 128 == 0:
                continue
            one = ctx.solve(psi, **kw)
            assert stats[k]["inner_iters_total"] == one.stats["inner_iters_total"]
            assert torch.equal(phis[k], one.phi), psi.shape
