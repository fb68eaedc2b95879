"""The even/odd MFMA DCT stages (mixed path, sides multiples of 128) on every
tile shape: fine below 128 tiles of 128 x 128 in the launch, narrow, wide in the
first three stages from 576 and in all from 1024; sides that are odd multiples
of 128, where a wide tile has no right partner.  Reference: dense transforms in
FP64; tolerances those of the other DCT applies, relative to max |s| (split bf16
2e-4, scaled fp16 1e-2).  The shape is chosen by the launch, so a map's result in
a batch that takes wide tiles equals its single solve on fine ones bit for bit.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(128, 128), (128, 384), (640, 128), (1024, 896), (1024, 1920), (1408, 1664), (3200, 3072),
         (3072, 3200), (4224, 4096), (4096, 4224)]


def dct_matrix(n):
    k = torch.arange(n, device="cuda", dtype=torch.float64)
    c = torch.cos(math.pi * k[:, None] * (2 * k[None, :] + 1) / (2 * n)) * math.sqrt(2.0 / n)
    c[0] = math.sqrt(1.0 / n)
    return c


@pytest.mark.parametrize("mode,rel", [("split_bf16", 2e-4), ("fp16_scaled", 1e-2)])
@pytest.mark.parametrize("M,N", SIZES)
def test_dct_even_odd(mode, rel, M, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if mode == "split_bf16" and M * N > 5_000_000:
        pytest.skip("the split takes no wide tiles")
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


@pytest.mark.parametrize("large", [1, 2, 4])
def test_dct_even_odd_batch_matches_single(large):
    """Launches of 339, 595 and 1107 tiles (narrow, wide but for the last stage,
    wide) against the single solves (fine, and narrow for the large map)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    rng = np.random.default_rng(7)
    shapes = [(128, 384), (384, 640), (1024, 1024)] + [(2048, 2048)] * large
    psis = [torch.from_numpy(rng.uniform(-3.0, 3.0, s)).cuda() for s in shapes]
    kw = dict(p=0.0, preconditioner="dct", precision="mixed", dct_mode="fp16_scaled", k_max=1,
              outer_tol=0.0)
    with Context(0) as ctx:
        phis, _, stats = ctx.batch(psis, **kw)
        for k, psi in enumerate(psis[:4]):
            one = ctx.solve(psi, **kw)
            assert stats[k]["inner_iters_total"] == one.stats["inner_iters_total"]
            assert torch.equal(phis[k], one.phi), psi.shape
