"""The bounded wait of the natural-order sweeps: made to give up at the first value
that is not there yet, the strips below the first do so (nothing hangs, every kernel
ends), and each call says so; with the default bound back everything is as before."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("pc", ["ilu0", "ssor"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_a_lost_wait_is_reported(precision, pc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_13675_amd import binding
    dtype = np.float64 if precision == "fp64" else np.float32
    rng = np.random.default_rng(2)
    M, N = 640, 200
    U, V = (rng.uniform(0.01, 1.0, (M, N)).astype(dtype) for _ in range(2))
    U[:, -1] = 0.0
    V[-1] = 0.0
    U, V, r = dev(U), dev(V), dev(rng.standard_normal((M, N)).astype(dtype))
    psi = dev(rng.uniform(-3.0, 3.0, (M, N)))
    kw = dict(preconditioner=pc, precision=precision, k_max=1, l_max=10, outer_tol=0.0, check=False,
              max_refine=1)
    with binding.Context(0) as ctx:
        want = ctx.precond_apply(U, V, r, pc, precision=precision)
        phi = ctx.solve(psi, **kw)
        piv = ctx.ilu_pivots(U, V, precision=precision)
        ctx.debug_sweep_no_wait(True)
        with pytest.raises(binding.LpuError) as e:
            ctx.precond_apply(U, V, r, pc, precision=precision)
        assert e.value.code == binding.ERR_HIP and "gave up" in ctx.last_error()
        with pytest.raises(binding.LpuError):
            ctx.ilu_pivots(U, V, precision=precision)
        assert "gave up" in ctx.last_error()
        lost = ctx.solve(psi, **kw)
        assert lost.status == binding.ERR_BREAKDOWN and "gave up" in ctx.last_error()
        ctx.debug_sweep_no_wait(False)
        assert torch.equal(ctx.precond_apply(U, V, r, pc, precision=precision), want)
        assert torch.equal(ctx.ilu_pivots(U, V, precision=precision), piv)
        again = ctx.solve(psi, **kw)
        assert again.status == phi.status and torch.equal(again.phi, phi.phi)
