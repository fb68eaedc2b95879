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
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


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
