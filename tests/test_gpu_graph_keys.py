"""Captured iteration graphs are kept across calls under a key of what they
launch: a call whose launches differ from a kept graph's must not replay it."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_dct_grid_cap_takes_effect_after_a_capture():
    """1024 x 1024 in scaled fp16: 64 list entries of four fine tiles each.  A cap
    of 64 blocks makes every block walk four tiles one after another, so the
    solve takes about twice as long; with graphs of the other cap replayed it
    would take as long.  The phase does not depend on the cap."""
    from paper_2203_13675_amd.binding import Context
    psi = dev(np.random.default_rng(3).uniform(-3.0, 3.0, (1024, 1024)))
    out = torch.zeros_like(psi)
    kw = dict(p=0.0, preconditioner="dct", precision="mixed", dct_mode="fp16_scaled", k_max=1,
              outer_tol=0.0, check=False)

    def best(ctx, cap):
        ctx.set_tuning(dct_grid=cap)
        t = []
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            phi = ctx.solve(psi, phi=out, **kw).phi
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t), phi.clone()

    with Context(0) as ctx:
        wide, a = best(ctx, 2048)
        narrow, b = best(ctx, 64)
        again, c = best(ctx, 2048)
    assert torch.equal(a, b) and torch.equal(a, c)
    assert narrow > 1.3 * max(wide, again), (wide, narrow, again)


@pytest.mark.parametrize("dct_mode", ["fp32", "split_bf16"])
def test_batches_of_more_maps_on_the_same_grids(dct_mode):
    """Batches of two, three and five maps whose launches have the same grids, in
    one context: the FP32 transforms' finisher is a launch of one block per map,
    so a graph kept from two maps would never finish the third."""
    from paper_2203_13675_amd.binding import Context
    rng = np.random.default_rng(4)
    shapes = [[(200, 200)] * 2, [(200, 200), (96, 100), (90, 120)], [(200, 200)] + [(90, 60)] * 4]
    batches = [[dev(rng.uniform(-3.0, 3.0, s)) for s in b] for b in shapes]
    kw = dict(p=0.0, preconditioner="dct", precision="mixed", dct_mode=dct_mode, k_max=1,
              outer_tol=0.0, check=False)
    want = []
    for b in batches:
        with Context(0) as ctx:
            want.append(ctx.batch(b, **kw)[0])
    with Context(0) as ctx:
        ctx.batch([dev(rng.uniform(-3.0, 3.0, (220, 210)))] * 5, **kw)  # buffers that hold every batch
        for k in (0, 1, 2, 0):
            phis, _, _ = ctx.batch(batches[k], **kw)
            assert all(torch.equal(x, y) for x, y in zip(phis, want[k])), k
