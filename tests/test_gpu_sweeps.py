"""The natural-order sweeps (strips of 64 rows swept by one wave each, in
chunks of 16 steps) at the sizes where they can go wrong: rows around one and
two strips, columns around a chunk and a strip's skew, maps of a few pixels,
more strips than a launch has workgroups.  Reference: the oracle's CSR
factorisation in FP64 on the same (FP32-rounded for mixed) inputs.

Tolerances: FP64 1e-10 of max |s|, the bound of every other preconditioner
apply.  FP32: a solve with these weights (U, V in [0.01, 1]) is a recurrence
with row sums below 1, so its rounding errors of a few u32 per step are damped
and not accumulated; at most the condition of a strip of ~64 couplings, about
64 * 8 u32 = 3e-5, remains: 2e-4, the bound of the other FP32 sweep tests,
covers it.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = [(1, 1), (1, 2), (2, 1), (3, 1), (1, 17), (63, 16), (64, 15), (64, 79), (65, 1), (65, 64),
         (127, 33), (128, 129), (129, 80), (200, 161), (2, 700), (700, 2)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd.binding import Context
    c = Context(0)
    yield c
    c.close()


def system(M, N, seed, dtype=np.float64):
    rng = np.random.default_rng(seed)
    U = rng.uniform(0.01, 1.0, (M, N)).astype(dtype)
    V = rng.uniform(0.01, 1.0, (M, N)).astype(dtype)
    U[:, -1] = 0.0
    V[-1, :] = 0.0
    r = rng.standard_normal((M, N)).astype(dtype)
    if M * N == 1:
        r[:] = 0.0  # the only pixel is isolated
    return U, V, r


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precision,rel", [("fp64", 1e-10), ("mixed", 2e-4)])
@pytest.mark.parametrize("pc", ["ilu0", "ssor"])
@pytest.mark.parametrize("M,N", SIZES)
def test_sweep_edges(ctx, oracle, pc, precision, rel, M, N):
    U, V, r = system(M, N, M * 1000 + N, np.float64 if precision == "fp64" else np.float32)
    omega = 1.3 if pc == "ssor" else 1.0
    want = oracle.Preconditioner(pc, U.astype(np.float64), V.astype(np.float64),
                                 omega=omega).apply(r.astype(np.float64))
    got = ctx.precond_apply(dev(U), dev(V), dev(r), pc, precision=precision, omega=omega)
    err = np.abs(got.cpu().numpy() - want).max()
    assert err <= rel * (np.abs(want).max() + 1e-300), err


@pytest.mark.parametrize("precision,rel", [("fp64", 1e-10), ("mixed", 2e-4)])
def test_more_strips_than_workgroups(ctx, oracle, precision, rel):
    """520 strips in one map: the launch's workgroups take further strips by ticket."""
    U, V, r = system(520 * 64 - 7, 3, 5, np.float64 if precision == "fp64" else np.float32)
    want = oracle.Preconditioner("ssor", U.astype(np.float64), V.astype(np.float64)).apply(
        r.astype(np.float64))
    got = ctx.precond_apply(dev(U), dev(V), dev(r), "ssor", precision=precision)
    assert np.abs(got.cpu().numpy() - want).max() <= rel * np.abs(want).max()


@pytest.mark.parametrize("pc", ["ilu0", "ssor"])
def test_batch_of_many_strips_matches_single(ctx, pc):
    """A batch of more strips than workgroups, maps of one to five strips:
    every map's result equals its single solve bit for bit."""
    rng = np.random.default_rng(3)
    shapes = [(int(rng.integers(1, 300)), int(rng.integers(16, 90))) for _ in range(260)]
    assert sum(-(-m // 64) for m, _ in shapes) > 512
    psis = [dev(rng.uniform(-3.0, 3.0, s)) for s in shapes]
    kw = dict(p=0.0, preconditioner=pc, precision="mixed", k_max=1, outer_tol=0.0, l_max=12,
              max_refine=1)
    phis, _, stats = ctx.batch(psis, **kw)
    for k in range(0, len(shapes), 20):
        single = ctx.solve(psis[k], **kw)
        assert stats[k]["inner_iters_total"] == single.stats["inner_iters_total"], shapes[k]
        assert torch.equal(phis[k], single.phi), shapes[k]


def test_noalloc_sweep_under_capture():
    """The sweeps keep their counters and the launch count in device memory:
    a captured apply replayed on new inputs, with eager applies in between,
    gives the eager result every time."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd import binding
    stream = torch.cuda.Stream()
    with binding.Context(0, stream=stream) as c, torch.cuda.stream(stream):
        U, V, r = (dev(a) for a in system(200, 170, 8))
        s, e = torch.empty_like(r), torch.empty_like(r)
        apply = lambda out: c.precond_apply_noalloc(U, V, r, out, "ilu0")
        assert apply(e) == binding.OK
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            assert apply(s) == binding.OK
        for k in range(4):
            r.copy_(dev(system(200, 170, 20 + k)[2]))
            s.fill_(float("nan"))
            g.replay()
            assert apply(e) == binding.OK
            stream.synchronize()
            assert torch.equal(s, e), k
