"""Row products of more threads than one launch holds."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    import paper_2509_18497_amd as m
    return m


def test_bounce_of_more_threads_than_a_launch(g):
    """128 rows of 8.4 M coefficients, 64 threads to each 16 of a row: 2^32
    threads and some more.  E is a row's number times a column's pattern, F
    1/128 everywhere, so every sum is a whole number of 128ths below 2^24 and
    B is exact."""
    n, lights, K = 128, 524352, 16
    rp = torch.arange(0, n * n + 1, n, dtype=torch.int64, device="cuda")
    cols = torch.arange(n, dtype=torch.int32, device="cuda").repeat(n)
    ff = g.ff_from_csr(rp, cols, torch.full((n * n,), 1.0 / n, device="cuda"))
    pattern = (torch.arange(lights * K * 3, device="cuda") % 97).float()
    E = torch.empty((n, lights, K, 3), device="cuda")
    for i in range(n):
        torch.mul(pattern, float(i + 1), out=E[i].view(-1))
    rho = torch.full((n, 3), 0.5, device="cuda")
    B = torch.empty_like(E)
    g.transport_solve_noalloc(ff, rho, E, 1, B)
    for i in range(n):
        assert torch.equal(B[i].view(-1), pattern * (i + 1 + 0.5 * (n + 1) / 2)), i
    del E, B
    torch.cuda.empty_cache()
