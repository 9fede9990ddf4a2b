"""One sample per table at n = 128 with lists of more than 64 samples: every call that takes such an object."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,k,L", [(65, 128, 8), (96, 512, 32), (100, 60, 15), (127, 256, 8), (64, 128, 8)])
@pytest.mark.parametrize("N", [1, 130, 3000])
def test_calls(N, m, k, L):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_15479_amd as lsh
    n, w = 128, 4.0
    g = torch.Generator(device="cuda")
    g.manual_seed(m + N)
    data = torch.randn((N, n), generator=g, device="cuda")
    print(f"one sample per table: n=128 m={m} k={k} L={L} N={N}", flush=True)
    with lsh.LshParams(n, k, m, w, 5, shared_tables=L) as p:
        idx = torch.as_tensor(p.indices().astype("int64"), device="cuda").reshape(k, m)
        a = torch.zeros((k, n), dtype=torch.float64, device="cuda")
        a.scatter_add_(1, idx, torch.tensor(p.coeffs(), device="cuda").double().reshape(k, m))
        want, size = data.double() @ a.T, data.double().abs() @ a.abs().T
        got = lsh.project_fastlsh(p, data)
        assert ((got.double() - want).abs() <= 1e-5 * size).all()
        h = (want + torch.tensor(p.offsets(), device="cuda").double()) / w
        clear = (h - h.round()).abs() > 1e-4
        ids = lsh.hash_fastlsh(p, data)
        assert torch.equal(ids[clear], torch.floor(h)[clear].int())
        if (k // L) & (k // L - 1) == 0:
            assert torch.equal(lsh.hash_fastlsh_keys(p, data, L), lsh.pack_keys(p, ids, L))
            both = lsh.hash_fastlsh_ids_keys(p, data, L)
            assert torch.equal(both[0], ids) and torch.equal(both[1], lsh.pack_keys(p, ids, L))
        lsh.hash_signs(p, data)
        kappa2 = lsh.mips_kappa(p, data)
        exact = torch.stack([(data[:, idx[l * (k // L)]].double() ** 2).sum(1).max() for l in range(L)])
        assert torch.allclose(kappa2.double(), exact, rtol=2e-6)
        norms = torch.stack([(data[:, idx[l * (k // L)]].double() ** 2).sum(1) for l in range(L)], 1).repeat_interleave(k // L, 1)
        a0 = torch.tensor(p.mips_coeffs(), device="cuda").double()
        lift = (kappa2.double().repeat_interleave(k // L) - norms).clamp(min=0).sqrt()
        h = (want + a0 * lift + torch.tensor(p.offsets(), device="cuda").double()) / w
        clear = ((h - h.round()).abs() > 1e-3) & (lift > 0.1)
        assert torch.equal(lsh.hash_mips_data(p, data, kappa2)[clear], torch.floor(h)[clear].int())
        lsh.hash_mips_query(p, data)
