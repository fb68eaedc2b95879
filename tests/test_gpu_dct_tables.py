"""The DCT tables, filled on the device, through the FP64 apply of a one-row or
one-column map: one pixel, sides around the 64 columns that rows are padded to
and around the block layout's 128, a long side (k (2j + 1) far beyond 2^24).

Reference: the transform in long double with angles reduced mod 2 pi.  Every
table entry is within u of its value and each of the two transforms is a sum of
n products, so the result is within 4 n u ||r|| / lambda_min in the 2-norm.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("column", [False, True])
@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 127, 128, 256, 1500, 4096])
def test_dct_tables(n, column):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    rng = np.random.default_rng(n)
    r = rng.standard_normal(n)
    shape = (n, 1) if column else (1, n)
    U = np.zeros(shape)
    V = np.zeros(shape)
    (V if column else U).reshape(-1)[:-1] = 1.0
    with Context(0) as ctx:
        s = ctx.precond_apply(torch.from_numpy(U).cuda(), torch.from_numpy(V).cuda(),
                              torch.from_numpy(r.reshape(shape)).cuda(), "dct", precision="fp64")
    s = s.cpu().numpy().reshape(-1)
    pi = np.arctan(np.longdouble(1)) * 4
    q = np.cos(pi * np.arange(4 * n) / (2 * n)) * np.sqrt(np.longdouble(2) / n)
    k = np.arange(n, dtype=np.int64)
    C = q[(k[:, None] * (2 * k[None, :] + 1)) % (4 * n)]
    C[0] = np.sqrt(np.longdouble(1) / n)
    lam = 2 - 2 * np.cos(pi * k / n)
    x = C @ r.astype(np.longdouble)
    x[1:] /= lam[1:]
    x[0] = 0
    want = C.T @ x
    err = float(np.linalg.norm((s - want).astype(np.float64)))
    assert err <= 4 * n * 2.0 ** -53 * np.linalg.norm(r) / float(lam[1])
