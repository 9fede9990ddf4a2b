"""The largest norms of a large data set are taken by waves that hold several tables' lists, those of a small
one by waves that hold one: the same numbers, bit for bit (the data hash relies on it)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,k,m,L", [
    (960, 1024, 128, 64),    # four tables a wave
    (500, 800, 100, 40),     # two blocks of functions a table, the last waves idle
    (260, 136, 65, 34),      # tables of four functions, two and a bit for every wave
    (964, 128, 90, 16),      # one table a wave already
    (500, 640, 100, 32),     # two tables a wave
    (960, 80, 128, 20),      # the same, the last waves with one table and none
])
def test_kappa_of_all_equals_largest_of_parts(n, k, m, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_15479_amd as lsh
    N = 40000
    g = torch.Generator(device="cuda")
    g.manual_seed(n + m)
    data = torch.randn((N, n), generator=g, device="cuda")
    with lsh.LshParams(n, k, m, 4.0, 3, shared_tables=L) as p:
        print(f"kappa n={n} k={k} m={m} L={L}", flush=True)
        whole = lsh.mips_kappa(p, data)
        parts = torch.stack([lsh.mips_kappa(p, data[i:i + 480].clone()) for i in range(0, N, 480)])
        assert torch.equal(whole, parts.max(dim=0).values)
        idx = torch.as_tensor(p.indices().astype("int64"), device="cuda").reshape(L, k // L, m)[:, 0]
        exact = torch.stack([(data[:, idx[l]].double() ** 2).sum(1).max() for l in range(L)])
        assert torch.allclose(whole.double(), exact, rtol=2e-6)
