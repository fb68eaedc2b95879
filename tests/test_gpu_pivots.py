"""The no-fill pivots p = a - U_W^2 / p_W - V_N^2 / p_N bit for bit against a plain
factorisation whose quotients are IEEE divisions (numpy, the same order of
operations), for couplings of every size: ordinary weights, weights over many
decades, zeros (also along a strip's edge), and couplings so small or large that
squares, pivots or their reciprocals leave the normal range.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def plain_pivots(U, V):
    T = U.dtype.type
    M, N = U.shape
    uw, vn = np.zeros_like(U), np.zeros_like(V)
    uw[:, 1:], vn[1:] = U[:, :-1], V[:-1]
    with np.errstate(all="ignore"):
        a = ((uw + U) + vn) + V
        p = np.ones((M + 1, N + 1), U.dtype)  # p[i + 1, j + 1]
        for d in range(M + N - 1):
            i = np.arange(max(0, d - N + 1), min(M, d + 1))
            j = d - i
            w, n, v = uw[i, j], vn[i, j], a[i, j].copy()
            v = np.where(w != 0, v - (w * w) / p[i + 1, j], v)
            v = np.where(n != 0, v - (n * n) / p[i, j + 1], v)
            v = np.where(v < T(1e-4) * a[i, j], a[i, j], v)
            p[i + 1, j + 1] = np.where(a[i, j] == 0, T(1), v)
    return p[1:, 1:]


def couplings(kind, M, N, dtype, rng):
    tiny = np.finfo(dtype).tiny
    big = np.sqrt(np.finfo(dtype).max)
    if kind == "ordinary":
        f = lambda: rng.uniform(0.01, 1.0, (M, N))
    elif kind == "decades":  # Eq. (6) at p = 0 over residuals of 1e-3 to 1e5
        f = lambda: 0.01 / (10.0 ** rng.uniform(-6, 10, (M, N)) + 0.01)
    elif kind == "zeros":
        f = lambda: rng.uniform(0.01, 1.0, (M, N)) * (rng.random((M, N)) < 0.6)
    elif kind == "tiny":  # about and below the smallest normal number
        f = lambda: rng.uniform(0.2, 3.0, (M, N)) * tiny * 10.0 ** rng.uniform(-4, 1, (M, N))
    elif kind == "huge":  # squares overflow
        f = lambda: rng.uniform(0.2, 3.0, (M, N)) * big * 10.0 ** rng.uniform(-1, 2, (M, N))
    elif kind == "top":  # diagonals overflow here and there
        f = lambda: np.where(rng.random((M, N)) < 0.02, 0.9 * np.finfo(dtype).max, rng.uniform(0.01, 1.0, (M, N)))
    else:  # "mixed": ordinary ones, with a few extreme ones and zeros among them
        def f():
            x = rng.uniform(0.01, 1.0, (M, N))
            k = rng.integers(0, 400, (M, N))
            x[k == 0], x[k == 1], x[k == 2], x[k == 3] = 0.0, 2.5 * tiny, tiny / 8, big
            return x
    U, V = f().astype(dtype), f().astype(dtype)
    U[:, -1] = 0.0
    V[-1] = 0.0
    if kind == "zeros" and M > 64:
        V[63] = 0.0  # no coupling across the first strip's edge
    return U, V


@pytest.mark.parametrize("M,N", [(1, 200), (64, 70), (65, 33), (200, 161), (150, 400)])
@pytest.mark.parametrize("kind", ["ordinary", "decades", "zeros", "tiny", "huge", "top", "mixed"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_pivots_are_those_of_plain_divisions(precision, kind, M, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    dtype = np.float64 if precision == "fp64" else np.float32
    rng = np.random.default_rng(M * 1000 + N)
    U, V = couplings(kind, M, N, dtype, rng)
    want = plain_pivots(U, V)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    with Context(0) as ctx:
        got = ctx.ilu_pivots(dev(U), dev(V), precision=precision).cpu().numpy()
    same = (got == want) | (np.isnan(got) & np.isnan(want))
    assert same.all(), (int((~same).sum()), got[~same][:4], want[~same][:4])
