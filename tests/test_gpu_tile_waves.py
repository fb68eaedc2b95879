"""The stencil tiles (128 columns by tile_rows rows, four rows to a wave, up to
eight waves to a tile) at the sizes where they can go wrong: rows around a
wave's four, a tile's edge and a second turn of the waves; columns around a
half and a whole tile; one pixel, one row, one column.

apply_A: |err| <= 16 u |A| |x| entrywise (nine products and sums, each rounded
once), the bound of the other operator tests.

Solves: p = 2 makes every weight the same c, so the exact solution is the
inverse Neumann Laplacian (the oracle's DCT) of D^T Delta.  A solve that stops at
||r|| <= tol ||b|| is off by at most tol ||b|| / lambda_min in the 2-norm with
lambda_min = 2 - 2 cos(pi / max(M, N)) (c cancels), plus rounding of the
accumulated FP64 iterate, below 1e-12 of it per unit of condition
8 / lambda_min.  The refined residual is formed in FP64, so the bound holds for
both precisions.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U64, U32 = 2.0 ** -53, 2.0 ** -24
SIZES = [(1, 1), (1, 129), (3, 64), (4, 65), (5, 127), (7, 128), (8, 130), (15, 1), (16, 63),
         (17, 129), (31, 2), (33, 257), (63, 66), (65, 128), (100, 40)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    c = Context(0)
    yield c
    c.close()


def dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


@pytest.mark.parametrize("rows", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("M,N", SIZES)
def test_tile_waves(ctx, oracle, M, N, rows):
    ctx.set_tuning(tile_rows=rows)
    rng = np.random.default_rng(1000 * M + N)
    U = rng.uniform(0.01, 1.0, (M, N))
    V = rng.uniform(0.01, 1.0, (M, N))
    U[:, -1] = 0.0
    V[-1, :] = 0.0
    x = rng.standard_normal((M, N))
    for prec, t, u in (("fp64", np.float64, U64), ("mixed", np.float32, U32)):
        Ut, Vt, xt = (a.astype(t) for a in (U, V, x))
        U6, V6, x6 = (a.astype(np.float64) for a in (Ut, Vt, xt))
        want = oracle.apply_A(U6, V6, x6)
        # |A| |x|: A has a positive diagonal and negative couplings
        scale = 2 * oracle.diag_A(U6, V6) * np.abs(x6) - oracle.apply_A(U6, V6, np.abs(x6))
        got = ctx.apply_A(dev(Ut, t), dev(Vt, t), dev(xt, t), prec).cpu().numpy()
        assert np.all(np.abs(got - want) <= 16 * u * scale), (prec, "apply_A")
    if M * N == 1:
        return
    psi = rng.uniform(-np.pi, np.pi, (M, N))
    dx, dy = oracle.wrapped_differences(psi)
    one = np.ones((M, N))
    U1, V1 = one.copy(), one.copy()
    U1[:, -1] = 0.0
    V1[-1, :] = 0.0
    b = oracle.rhs(U1, V1, dx, dy)
    exact = oracle.Preconditioner("dct", U1, V1).apply(b)
    exact -= exact.mean()
    lmin = 2.0 - 2.0 * np.cos(np.pi / max(M, N))
    tol = 1e-9
    bound = tol * np.linalg.norm(b) / lmin + 1e-12 * 8 / lmin * np.linalg.norm(exact)
    for prec in ("fp64", "mixed"):
        for pc in ("none", "jacobi", "ssor_rb"):
            res = ctx.solve(dev(psi, np.float64), p=2.0, preconditioner=pc, tol=tol, precision=prec)
            phi = res.phi.cpu().numpy()
            err = np.linalg.norm(phi - phi.mean() - exact)
            assert res.stats["final_relres"] <= tol, (prec, pc)
            assert err <= bound, (prec, pc, err, bound)
