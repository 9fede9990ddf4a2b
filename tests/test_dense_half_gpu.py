"""The dense product from two-way fp16 splits (sums of 128 terms and more, n other than 128) against the
same sums in 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lsh():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_15479_amd as lib
    lib.load_library()
    return lib


def _exact(p, data):
    a = torch.tensor(p.coeffs(), device="cuda").double().reshape(p.k, p.n)
    return data.double() @ a.T, data.double().abs() @ a.abs().T


def _data(kind, N, n):
    g = torch.Generator(device="cuda")
    g.manual_seed(N * 31 + n)
    x = torch.randn((N, n), generator=g, device="cuda")
    at = torch.arange(n, device="cuda")
    if kind == "late":        # nothing in the coordinates a scale is first taken from, but for some vectors
        x = x * (at >= n - 17) * (torch.arange(N, device="cuda")[:, None] % 7 != 3)
    elif kind == "rise":      # the last coordinates leave the range the first ones suggest
        x = x * torch.where(at >= n - 17, 1e4, 1e-3)
    elif kind == "fall":
        x = x * torch.where(at >= 16, 1e-5, 1.0)
    elif kind == "rows":      # every vector of another size
        x = x * torch.exp(20.0 * torch.randn((N, 1), generator=g, device="cuda"))
    elif kind == "tiny":
        x = x * 1e-37
    elif kind == "huge":
        x = x * 1e35
    return x


@pytest.mark.parametrize("kind", ["normal", "late", "rise", "fall", "rows", "tiny", "huge"])
@pytest.mark.parametrize("N,n,k", [(1, 132, 64), (257, 148, 250), (300, 960, 260), (255, 1028, 512)])
def test_projections(lsh, kind, N, n, k):
    """Off by at most 2^-21 of sum |a_i v_i| by the split (2^-23 for each operand, and 2^-22 for the product of the
    low terms, which is left out) and n / 16 * 3 roundings of 2^-24 (the accumulation, one for sixteen terms and
    product, all of them at the largest partial sum): 1.1e-5 at n = 960 in the worst case, a thirtieth of that as seen.
    The bound here is 2e-6, which an fp32 sum of these distributions keeps to."""
    data = _data(kind, N, n)
    print(f"dense fp16 product: {kind} N={N} n={n} k={k}", flush=True)
    with lsh.LshParams(n, k, n, 4.0, 11) as p:
        want, size = _exact(p, data)
        got = lsh.project_e2lsh(p, data).double()
        p.set_dense_arithmetic(lsh.DENSE_FP32)
        plain = lsh.project_e2lsh(p, data).double()
    worst = ((got - want).abs() / size.clamp(min=1e-300)).max().item()
    assert worst < 2e-6, worst
    assert (got - want).norm().item() <= 1.5 * (plain - want).norm().item()


def test_ids_do_not_depend_on_the_batch(lsh):
    """A vector's scale is its own: its ids are the same alone, among others, and beside vectors that are
    contracted apart or hold no number at all."""
    n, k = 964, 300
    data = _data("normal", 600, n)
    with lsh.LshParams(n, k, n, 3.0, 12) as p:
        ids = lsh.hash_e2lsh(p, data)
        assert torch.equal(lsh.hash_e2lsh(p, data[100:101].clone()), ids[100:101])
        assert torch.equal(lsh.hash_e2lsh(p, data[37:400].clone()), ids[37:400])
        odd = data.clone()
        odd[::5] = _data("rise", 120, n)
        odd[3] = float("inf")
        odd[7] = float("nan")
        odd[11] = 0.0
        got = lsh.hash_e2lsh(p, odd)
        same = torch.ones(600, dtype=torch.bool, device="cuda")
        same[::5] = False
        same[[3, 7, 11]] = False
        assert torch.equal(got[same], ids[same])
        off = torch.tensor(p.offsets(), device="cuda")
        assert torch.equal(got[11], torch.floor(off / 3.0).int())


@pytest.mark.parametrize("N,n,k,w", [(40000, 132, 250, 4.0), (15000, 964, 640, 3.0), (12000, 980, 900, 8.0)])
def test_few_vectors_equal_many(lsh, N, n, k, w):
    """Few vectors take a kernel of their own: the same numbers, whatever the vectors' scales."""
    data = _data("normal", N, n)
    for i, kind in enumerate(("late", "rise", "fall", "rows", "tiny", "huge")):
        data[i::11] = _data(kind, N, n)[i::11]
    with lsh.LshParams(n, k, n, w, 13) as p:
        print(f"dense fp16 product, few against many: n={n} k={k}", flush=True)
        ids, proj = lsh.hash_e2lsh(p, data), lsh.project_e2lsh(p, data)
        for first, count in ((0, 1), (31, 33), (N - 257, 257), (5000, 2000)):
            part = data[first:first + count].clone()
            assert torch.equal(lsh.project_e2lsh(p, part), proj[first:first + count])
            assert torch.equal(lsh.hash_e2lsh(p, part), ids[first:first + count])


@pytest.mark.parametrize("n,k,m,again", [(960, 250, 128, False), (1028, 512, 300, True), (132, 500, 128, False)])
@pytest.mark.parametrize("large", [1e6, 1e10, 1e30])
def test_unsampled_coordinates_have_no_influence(lsh, n, k, m, again, large):
    """Eq. 5 depends on the m coordinates that a function samples alone, also where it runs as a dense product
    over all n: a large coordinate changes no bit of the functions that do not sample it."""
    N = 300
    data = _data("normal", N, n)
    at = n // 2
    spoilt = data.clone()
    spoilt[:, at] = large
    with lsh.LshParams(n, k, m, 4.0, 17, with_replacement=again) as p:
        idx = torch.as_tensor(p.indices().astype("int64"), device="cuda").reshape(k, m)
        without = ~(idx == at).any(1)
        assert without.any()
        p.set_dense_arithmetic(lsh.DENSE_MATRIX)
        print(f"dense product of a sampled object: n={n} k={k} m={m} large={large}", flush=True)
        assert torch.equal(lsh.project_fastlsh(p, spoilt)[:, without], lsh.project_fastlsh(p, data)[:, without])
        assert torch.equal(lsh.hash_fastlsh(p, spoilt)[:, without], lsh.hash_fastlsh(p, data)[:, without])
        a = torch.zeros((k, n), dtype=torch.float64, device="cuda")
        a.scatter_add_(1, idx, torch.tensor(p.coeffs(), device="cuda").double().reshape(k, m))
        want, size = spoilt.double() @ a.T, spoilt.double().abs() @ a.abs().T
        worst = ((lsh.project_fastlsh(p, spoilt).double() - want).abs() / size).max().item()
        assert worst < 1e-5, worst


def _odd(kind, N, n):
    """Vectors that few of their coordinates carry."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N * 17 + n)
    x = torch.randn((N, n), generator=g, device="cuda")
    at = torch.randint(0, n, (N, 1), generator=g, device="cuda")
    if kind == "one":
        return torch.zeros_like(x).scatter_(1, at, torch.exp2(torch.round(3 * x[:, :1])))
    if kind == "sparse":
        return x * (torch.rand((N, n), generator=g, device="cuda") < 5.0 / n)
    if kind == "small beside one":
        return x.scatter_(1, at, 1e10)
    if kind == "powers":       # every coordinate of another size
        return x * torch.exp(40.0 * torch.randn((N, n), generator=g, device="cuda")).clamp(1e-34, 1e30)
    if kind == "least":        # no scale takes these to the usual size
        return x * 2e-38
    if kind == "column":       # one column of another unit, not looked at for a scale; some vectors without it
        x[torch.arange(N, device="cuda") % 50 != 7, n // 2 + 5] *= 1e7
        return x
    if kind == "nearly all":
        x[torch.arange(N, device="cuda") % 23 != 5] = _odd("one", N, n)[torch.arange(N, device="cuda") % 23 != 5]
        return x
    assert kind == "mixed"
    x[::3] = _odd("one", N, n)[::3]
    x[1::37] = _odd("small beside one", N, n)[1::37]
    x[2::41] = 0.0
    return x


@pytest.mark.parametrize("kind", ["one", "sparse", "small beside one", "powers", "least", "column", "nearly all", "mixed"])
@pytest.mark.parametrize("N,n,k,w", [(20000, 960, 1024, 4.0), (3000, 4096, 2048, 3.0), (700, 260, 250, 3.0), (150001, 260, 250, 4.0)])
def test_vectors_of_few_coordinates(lsh, kind, N, n, k, w):
    """A function may give such a vector's largest coordinates small coefficients: all that the splits lose must stay
    below 1e-5 of that small sum of |a_i v_i| too, for every function and vector.  (Without products of their own
    they are off by up to 2e-5 of it here.)  The same numbers in a launch of few vectors and of many, and beside
    other vectors; of a single coordinate, a power of two here, the product itself."""
    data = _odd(kind, N, n)
    print(f"dense fp16 product, vectors of few coordinates: {kind} N={N} n={n} k={k}", flush=True)
    with lsh.LshParams(n, k, n, w, 19) as p:
        got, ids = lsh.project_e2lsh(p, data), lsh.hash_e2lsh(p, data)
        for i in range(0, N, 4000):
            want, size = _exact(p, data[i:i + 4000])
            worst = ((got[i:i + 4000].double() - want).abs() / size.clamp(min=1e-300)).max().item()
            assert worst < 1e-5, worst
            if kind == "one":
                assert torch.equal(got[i:i + 4000], want.float())
            off = torch.tensor(p.offsets(), device="cuda").double()
            edge = ((want + off) / w) - ((want + off) / w).round()
            clear = (edge.abs() > 1e-4 + 1e-5 * size / w) & (want.abs() / w < 2e9)
            assert torch.equal(ids[i:i + 4000][clear], torch.floor((want + off) / w)[clear].int())
        for first, count in ((0, 1), (31, 33), (N - 257, 257), (5, 64)):
            part = data[first:first + count].clone()
            assert torch.equal(lsh.project_e2lsh(p, part), got[first:first + count])
            assert torch.equal(lsh.hash_e2lsh(p, part), ids[first:first + count])


def test_bound_of_a_split(lsh):
    """Vectors made for one function each: the eight looked-at coordinates at which the split of the function's
    coefficient and of 1 + 2^-11 - 2^-21 + 2^-23 loses most, with the signs that add the losses up.  More than 2^-22 of the
    sum is lost, and no more than 2^-21 and the roundings of the accumulation (24 products of eight equal terms at
    most, each off by 2^-24 of the sum)."""
    import numpy as np
    n, k = 960, 512
    looked = np.concatenate([np.arange(48), np.arange(320, 336), np.arange(640, 656)])
    with lsh.LshParams(n, k, n, 4.0, 23) as p:
        a = p.coeffs().reshape(k, n).astype(np.float64)
        v = 1 + 2.0 ** -11 - 2.0 ** -21 + 2.0 ** -23
        assert np.float32(v) == v
        scaled = a * 2.0 ** (14 - np.floor(np.log2(np.abs(a).max(1, keepdims=True))))

        def terms(x):
            high = x.astype(np.float16).astype(np.float64)
            return high, (x - high).astype(np.float16).astype(np.float64)

        (a1, a2), (v1, v2) = terms(scaled), terms(np.float64(v * 32))
        loss = (a1 * v1 + a1 * v2 + a2 * v1 - scaled * v * 32) / np.abs(scaled * v * 32)
        data = np.zeros((k, n), dtype=np.float32)
        for j in range(k):
            at = looked[np.argsort(-np.abs(loss[j, looked]))[:8]]
            data[j, at] = v * np.sign(loss[j, at])  # the term is off by loss * |term|: signs that make all losses positive
        print("dense fp16 product: largest losses of a split", flush=True)
        got = lsh.project_e2lsh(p, torch.tensor(data, device="cuda")).cpu().numpy().astype(np.float64)
    exact = (data.astype(np.float64) * a).sum(1)
    off = (np.diagonal(got) - exact) / (np.abs(data) * np.abs(a)).sum(1)
    assert off.max() > 2.0 ** -22, off.max()
    assert np.abs(off).max() < 2.0 ** -21 + 24 * 2.0 ** -24, np.abs(off).max()
