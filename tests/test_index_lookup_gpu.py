"""Bucket lookup and the processing of candidates at the edges of their tiles: 8 lanes a lookup
or, for more than 16384 lookups, 2; 256 buckets at a time, lists of 1024 candidates, an LDS table of 2048 ids met before, vectors of
whole and of partial 16-byte pieces, the query in LDS or not."""
import numpy as np
import pytest

from oracle import index as oindex

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lsh():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2309_15479_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("N,L,distinct", [(1, 2, 1), (2, 2, 2), (3, 2, 1), (8, 2, 1), (9, 2, 9), (80, 2, 80), (81, 2, 40),
                                          (4624, 3, 300), (70001, 3, 70001), (70001, 2, 3)])
def test_probe_finds_both_ends_of_every_bucket(lsh, N, L, distinct):
    rng = np.random.default_rng(N + distinct)
    pool = rng.integers(0, 2 ** 64, size=(distinct, L), dtype=np.uint64)
    pool[0] = 0
    pool[-1] = 2 ** 64 - 1
    keys = np.take_along_axis(pool, rng.integers(0, distinct, size=(N, L)), axis=0)
    queries = np.concatenate([pool[:400], pool[:400] + np.uint64(1), pool[:400] - np.uint64(1)])
    many = np.concatenate([queries] * (1 + 16384 // queries.size))
    table = np.sort(keys, axis=0)
    with lsh.LshIndex(torch.as_tensor(keys.view(np.int64), device="cuda")) as ix:
        for asked in (queries, many):
            start, count = ix.probe(torch.as_tensor(asked.view(np.int64), device="cuda"))
            for l in range(L):
                first = np.searchsorted(table[:, l], asked[:, l], side="left")
                end = np.searchsorted(table[:, l], asked[:, l], side="right")
                assert np.array_equal(start[:, l].cpu().numpy().view(np.uint32), first), l
                assert np.array_equal(count[:, l].cpu().numpy().view(np.uint32), end - first), l


@pytest.mark.parametrize("N,L,Q", [(120001, 9, 1821), (132000, 8, 2049), (70001, 130, 128), (70100, 15, 1111), (48000, 23, 3000),
                                   (70001, 9, 1821), (66000, 8, 2049)])
def test_probe_table_after_table(lsh, N, L, Q):
    """Tables that are more than two L2s and many queries: a table's lookups together, eight tables dealt to the XCDs at a
    time and what is left over, one to seven, to all of them (the last two rows: tables too small for that)."""
    rng = np.random.default_rng(N + L)
    keys = rng.integers(0, 3 * N, size=(N, L)).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    asked = rng.integers(0, 3 * N, size=(Q, L)).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    table = np.sort(keys, axis=0)
    with lsh.LshIndex(torch.as_tensor(keys.view(np.int64), device="cuda")) as ix:
        start, count = (t.cpu().numpy().view(np.uint32) for t in ix.probe(torch.as_tensor(asked.view(np.int64), device="cuda")))
    for l in range(L):
        first = np.searchsorted(table[:, l], asked[:, l], side="left")
        assert np.array_equal(start[:, l], first), l
        assert np.array_equal(count[:, l], np.searchsorted(table[:, l], asked[:, l], side="right") - first), l


# n: fewer pieces than a group of 8 lanes, partial pieces, several turns of a wave, around and above
# the largest query kept in LDS; Q on each side of 256, 768 and 1024 queries, soon done or not
@pytest.mark.parametrize("n,N,L,Q,distinct,shift", [(4, 50, 1, 3, 7, 0), (24, 5000, 3, 257, 4, 0), (30, 3000, 5, 20, 2, 0),
                                                    (24, 500, 2, 1001, 9, 0), (260, 300, 2, 769, 5, 0), (260, 300, 2, 1025, 5, 0), (128, 2500, 300, 9, 50, 0), (128, 400, 6, 5, 3, 1),
                                                    (960, 1500, 40, 30, 12, 0), (11264, 60, 3, 4, 3, 0),
                                                    (11268, 60, 3, 4, 3, 0), (16367, 40, 2, 3, 2, 0)])
@pytest.mark.parametrize("limit", [0, 1, 96, 1100])
def test_nearest_and_best_inner_product(lsh, n, N, L, Q, distinct, shift, limit):
    """Whole numbers from -8 to 8: every distance and inner product is below 2^24, so it is exact in
    any order of the sum and the smaller id of a tie has to win.  shift: vectors and queries start
    off a 16-byte boundary."""
    rng = np.random.default_rng(n + L + limit)
    data = rng.integers(-8, 9, size=(N, n)).astype(np.float32)
    data[N // 2:] = data[:N - N // 2]  # every vector twice: ties
    queries = rng.integers(-8, 9, size=(Q, n)).astype(np.float32)
    queries[0] = data[N - 1]
    keys = rng.integers(0, distinct, size=(N, L)).astype(np.uint64)
    qkeys = rng.integers(0, distinct + 1, size=(Q, L)).astype(np.uint64)
    qkeys[-1] = distinct  # no candidate

    def place(a):
        flat = torch.empty(a.size + shift, device="cuda")
        flat[shift:] = torch.as_tensor(a.reshape(-1), device="cuda")
        return flat[shift:].view(a.shape)

    with lsh.LshIndex(torch.as_tensor(keys.view(np.int64), device="cuda")) as ix:
        start, count = ix.probe(torch.as_tensor(qkeys.view(np.int64), device="cuda"))
        best, dist = ix.nearest(place(data), place(queries), start, count, max_candidates=limit)
        bip, ip = ix.best_inner_product(place(data), place(queries), start, count, max_candidates=limit)
        best, dist, bip, ip = (t.cpu().numpy() for t in (best, dist, bip, ip))
    buckets = oindex.probe(oindex.build(keys), qkeys)
    for q in range(Q):
        cand = oindex.candidates(buckets[q])
        cand = np.unique(np.asarray(cand[:limit] if limit else cand, dtype=np.int64))
        if not cand.size:
            assert best[q] == -1 and dist[q] == np.inf and bip[q] == -1 and ip[q] == -np.inf
            continue
        d = ((data[cand] - queries[q]) ** 2).sum(axis=1, dtype=np.float64)
        p = (data[cand] * queries[q]).sum(axis=1, dtype=np.float64)
        assert best[q] == cand[np.argmin(d)] and dist[q] == d.min()
        assert bip[q] == cand[np.argmax(p)] and ip[q] == p.max()
