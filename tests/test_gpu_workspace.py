"""A context's work buffers: what lp_unwrap_create reserves, and that calls of
several sizes leave them where they are.  Free device memory is compared before
and after calls whose buffers, allocated for themselves, would differ by tens of
MiB; the graphs are switched off and the DCT tables made beforehand, since both
take memory of their own.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SLACK = 4 << 20


def free_memory():
    """Free device memory, and what torch's own allocator holds."""
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0] + torch.cuda.memory_reserved()


def field(M, N, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(M, N, device="cuda", dtype=torch.float64, generator=g) * 6.0 - 3.0


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


KW = dict(p=0.0, preconditioner="dct", k_max=1, l_max=6, outer_tol=0.0, check=False, max_refine=1)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_reserved_context_solves_smaller_maps_in_place(precision):
    """480 x 448 takes more (smaller) DCT tiles than the 768 x 768 map reserved for."""
    from paper_2203_13675_amd.binding import Context
    psi, out = field(480, 448, 1), torch.zeros(480, 448, device="cuda", dtype=torch.float64)
    warm = [field(480, 64, 2), field(448, 64, 3)]  # the tables of both sides
    with Context(0, max_rows=768, max_cols=768) as c:
        c.set_tuning(use_graph=0)
        for w in warm:
            c.solve(w, precision=precision, **KW)
        before = free_memory()
        c.solve(psi, phi=out, precision=precision, **KW)
        assert abs(free_memory() - before) <= SLACK


@pytest.mark.parametrize("precision,sizes", [
    ("fp64", [(1024, 1024), (768, 768)]),    # 256 and 576 DCT tiles
    ("mixed", [(800, 1000), (480, 640)]),    # 208 and 300
])
def test_alternating_sizes_keep_the_buffers(precision, sizes):
    """The larger map takes fewer DCT tiles than the smaller one; after one call of
    each, neither allocates anything."""
    from paper_2203_13675_amd.binding import Context
    psis = [field(*s, 5) for s in sizes]
    outs = [torch.zeros_like(p) for p in psis]
    with Context(0) as c:
        c.set_tuning(use_graph=0)
        call = lambda k: c.solve(psis[k], phi=outs[k], precision=precision, **KW)
        call(0)
        call(1)
        call(0)
        before = free_memory()
        for k in (1, 0, 1):
            call(k)
            assert abs(free_memory() - before) <= SLACK, k


def test_precisions_and_batches_keep_the_buffers():
    """A large mixed batch, a small FP64 map, a wide flat map's sweep: the second
    turn allocates nothing, and the results are those of a context of one's own."""
    from paper_2203_13675_amd.binding import Context
    batch = [field(640, 512, k) for k in range(12)]
    small, flat = field(300, 200, 20), field(10, 40000, 21)
    kw = dict(KW, preconditioner="ssor")
    calls = [lambda c: c.batch(batch, precision="mixed", **KW)[0][3],
             lambda c: c.solve(small, precision="fp64", **KW).phi,
             lambda c: c.solve(flat, precision="fp64", **kw).phi]
    want = []
    for f in calls:
        with Context(0) as c:
            want.append(f(c))
    with Context(0) as c:
        c.set_tuning(use_graph=0)
        for f in calls * 2:
            f(c)
        before, got = free_memory(), []
        for k in (2, 0, 1, 0):
            got.append((k, calls[k](c)))
            assert abs(free_memory() - before) <= SLACK, k
    for k, phi in got:
        assert torch.equal(phi, want[k]), k
