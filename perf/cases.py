"""What the speed of this library is measured on: twelve uses of its public entry points.

A user hashes a data set once (ids, keys or both, sign words, the maximum-inner-product
hashes), builds an index from the keys, and then sends queries: few at a time where answers
are awaited, many at a time where they are collected.  The listed cases are one instance of
each, on the shapes this repository's workloads have (128, 960, 4096 and 16384 dimensions)
and on word-vector shapes (300 dimensions, sampling with replacement, a bucket width that is
no power of two, a number of vectors that fills no tile); draw() gives others of the same kinds.

Inputs are made on the GPU from the seed alone:
  bytes    integers in [0, 255] from a 100-cluster mixture (local image descriptors)
  unit     values in [0, 1] from a 1000-cluster mixture (global image descriptors)
  normal   independent N(0, 1) entries
  sphere   normal rows scaled to unit length
"""
import ctypes
import math

import torch

import paper_2309_15479_amd.binding as lsh

# The seed of the hash functions: a program draws them once and hashes all of its data with them.
FUNCTIONS_SEED = 7


def listed():
    return [
        # One search request at the moment it arrives: a handful of descriptors, hashed, looked
        # up in 32 tables and compared with the first 3 L candidates (the approximate version).
        dict(name="query_online", kind="query", dist="bytes", N=200_000, Q=8, n=128, k=512, m=32, L=32, w=512.0,
             limit=96),
        # A batch of requests against global descriptors, every candidate evaluated (the exact
        # version); about 480 candidates a query, most of them met in several tables.
        dict(name="query_batch", kind="query", dist="unit", N=100_000, Q=1000, n=960, k=1024, m=128, L=64, w=4.0,
             limit=0),
        # The hash codes alone of a request in 4096 dimensions, for tables that live elsewhere.
        dict(name="query_keys_wide", kind="hash", out="keys", dist="normal", N=100, n=4096, k=2048, m=64, L=128, w=8.0,
             shared=False, again=False),
        # A small collection: the launch is as short as its fixed costs.
        dict(name="ids_tiny", kind="hash", out="ids", dist="normal", N=10_000, n=128, k=64, m=32, L=8, w=4.0,
             shared=False, again=False),
        # Filling an index while keeping the ids for re-ranking.
        dict(name="ids_keys_sift", kind="hash", out="both", dist="bytes", N=1_000_000, n=128, k=512, m=32, L=32, w=16.0,
             shared=False, again=False),
        # Word vectors: sampling with replacement as the paper draws it, m = 30 as in its
        # experiments, nothing a multiple of a tile.
        dict(name="ids_words", kind="hash", out="ids", dist="normal", N=400_001, n=300, k=250, m=30, L=25, w=2.5,
             shared=False, again=True),
        dict(name="ids_gist", kind="hash", out="ids", dist="unit", N=1_000_000, n=960, k=1024, m=128, L=64, w=1.0,
             shared=False, again=False),
        dict(name="ids_wide", kind="hash", out="ids", dist="normal", N=200_000, n=4096, k=2048, m=256, L=128, w=8.0,
             shared=False, again=False),
        # The dense comparison path.
        dict(name="dense_gist", kind="dense", out="ids", dist="unit", N=1_000_000, n=960, k=1024, m=960, L=64, w=1.0),
        # Sign words of normalised vectors (angular similarity).
        dict(name="signs_angular", kind="signs", dist="sphere", N=500_000, n=16384, k=4096, m=512),
        # Preparing data for maximum inner product search: the largest norm of every table, then the hashes.
        dict(name="mips_data", kind="mips", dist="unit", N=300_000, n=960, k=1024, m=128, L=64, w=4.0),
        # The tables of an index from the keys of its vectors.
        dict(name="index_build", kind="index", dist="bytes", N=1_000_000, n=128, k=512, m=32, L=32, w=512.0),
    ]


def _log(rng, low, high):
    return max(low, min(high, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def draw(rng):
    """Another case of the same kinds: one vector to a million, 24 to 16384 dimensions."""
    kind = rng.choice(("query", "hash", "hash", "hash", "dense", "signs", "mips", "index"))
    dist = rng.choice(("bytes", "unit", "normal"))
    n = rng.choice((_log(rng, 24, 16384), _log(rng, 24, 1024), 4 * _log(rng, 8, 1024), 128, 128, 300, 960))
    g = rng.choice((4, 8, 16, 16, 32))
    L = _log(rng, 2, 64)
    m = min(n - 1, rng.choice((_log(rng, 8, 512), 30, 32, 64, 128)))
    # the deviation of a difference of projections within a cluster (or of near copies) is about
    # spread sqrt(m); the width is a few of those, a power of two or not
    spread = {"bytes": 28.0, "unit": 0.07, "normal": 1.4}[dist]
    w = spread * math.sqrt(m) * rng.uniform(0.5, 4.0)
    if rng.random() < 0.5:
        w = 2.0 ** round(math.log2(w))
    w = float("%.3g" % w)
    if kind == "query":
        n = min(n, 4096)
        m = min(m, n - 1)
        N = _log(rng, 1000, min(300_000, (1 << 28) // n))
        return dict(kind=kind, dist=dist, N=N, Q=_log(rng, 1, 4000), n=n, k=L * g, m=m, L=L, w=w, limit=3 * L)
    if kind == "index":
        n = min(n, 1024)
        m = min(m, n - 1)
        return dict(kind=kind, dist=dist, N=_log(rng, 1000, min(32_000_000 // L, (1 << 30) // n)), n=n, k=L * g, m=m, L=L, w=w)
    if kind == "dense":
        k = rng.choice((L * g, _log(rng, 16, 2048)))
        k = min(k, (1 << 22) // n)
        N = _log(rng, 1, min(1_000_000, (1 << 30) // n, (1 << 30) // k))
        return dict(kind=kind, out=rng.choice(("ids", "ids", "project")), dist=dist, N=N, n=n, k=k, m=n, L=1, w=w)
    if kind == "signs":
        k = 64 * L if rng.random() < 0.8 else _log(rng, 16, 2048)
        N = _log(rng, 1, min(1_000_000, (1 << 30) // n, (1 << 37) // (k * m)))
        return dict(kind=kind, dist="sphere", N=N, n=n, k=k, m=m)
    if kind == "mips":
        n = max(24, n // 4 * 4)
        m = min(m, n - 1)
        N = _log(rng, 1, min(1_000_000, (1 << 30) // n, (1 << 30) // (L * g)))
        return dict(kind=kind, dist=dist, N=N, n=n, k=L * g, m=m, L=L, w=w)
    out = rng.choice(("ids", "ids", "keys", "both", "project"))
    k = L * g if out in ("keys", "both") or rng.random() < 0.6 else _log(rng, 16, 2048)
    shared = k == L * g and rng.random() < 0.3
    N = _log(rng, 1, min(1_000_000, (1 << 30) // n, (1 << 30) // k, (1 << 38) // (k * m)))
    return dict(kind="hash", out=out, dist=dist, N=N, n=n, k=k, m=m, L=L if k == L * g else 1, w=w, shared=shared,
                again=rng.random() < 0.2)


def _rows(dist, N, n, gen):
    """[N, n] float32 on the GPU, made in blocks so that no second copy of the data is needed."""
    out = torch.empty((N, n), dtype=torch.float32, device="cuda")
    clusters, top, std = {"bytes": (100, 255.0, 20.0), "unit": (1000, 1.0, 0.05)}.get(dist, (0, 0.0, 1.0))
    if clusters:
        centres = torch.rand((clusters, n), generator=gen, device="cuda") * top
    step = max(1, (1 << 27) // n)
    for r in range(0, N, step):
        block = out[r:r + step]
        block.normal_(generator=gen)
        if clusters:
            which = torch.randint(0, clusters, (block.shape[0],), generator=gen, device="cuda")
            block.mul_(std).add_(centres[which])
            if dist == "bytes":
                block.round_()
            block.clamp_(0.0, top)
        elif dist == "sphere":
            block.div_(torch.linalg.vector_norm(block, dim=1, keepdim=True))
    return out


def _near_copies(data, Q, dist, gen):
    """Q queries: rows of the data with a little noise."""
    rows = torch.randint(0, data.shape[0], (Q,), generator=gen, device="cuda")
    noise = torch.empty((Q, data.shape[1]), device="cuda").normal_(generator=gen)
    out = data[rows] + noise * {"bytes": 2.0, "unit": 0.005}.get(dist, 0.1)
    if dist == "bytes":
        out = out.round_().clamp_(0.0, 255.0)
    return out


def _params(case):
    shared = case["L"] if case["kind"] == "mips" or case.get("shared") else 0
    return lsh.LshParams(case["n"], case["k"], case["m"], case.get("w", 1.0), FUNCTIONS_SEED,
                         with_replacement=case.get("again", False), shared_tables=shared)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    case = dict({"L": 1}, **case)
    params = _params(case)
    data = _rows(case["dist"], case["N"], case["n"], gen)
    state = {"case": case, "params": params, "data": data}
    if case["kind"] == "query":
        # the index lives on; what arrives is the queries
        keys = lsh.hash_fastlsh_keys(params, data, case["L"])
        state["index"] = lsh.LshIndex(keys)
        state["queries"] = _near_copies(data, case["Q"], case["dist"], gen)
    elif case["kind"] == "index":
        state["keys"] = lsh.hash_fastlsh_keys(params, data, case["L"])
        del state["data"]
    return state


class _Memory:
    """Device memory of an index, as torch.as_tensor takes it: the tensor holds this object, and
    this object the index, so the memory lives as long as the tensor."""

    def __init__(self, index, address, shape, kind):
        self.index = index
        self.__cuda_array_interface__ = {"data": (address, False), "shape": shape, "typestr": kind, "version": 2}


def _tables(index):
    """The sorted keys [L, N] and the ids in that order [L, N] of an index, in place."""
    keys, ids = ctypes.c_void_p(), ctypes.c_void_p()
    status = lsh.load_library().lsh_index_tables(index.handle, None, None, ctypes.byref(keys), ctypes.byref(ids))
    if status != lsh.LSH_OK:
        raise lsh.LshError(status, "lsh_index_tables")
    shape = (index.L, index.N)
    return (torch.as_tensor(_Memory(index, keys.value, shape, "<i8"), device="cuda"),
            torch.as_tensor(_Memory(index, ids.value, shape, "<i4"), device="cuda"))


def run(state):
    case, params = state["case"], state["params"]
    kind, L = case["kind"], case["L"]
    if kind == "query":
        index, queries = state["index"], state["queries"]
        keys = lsh.hash_fastlsh_keys(params, queries, L)
        start, count = index.probe(keys)
        best, distance = index.nearest(state["data"], queries, start, count, max_candidates=case["limit"])
        return {"keys": keys, "start": start, "count": count, "best": best, "distance": distance}
    if kind == "index":
        # a program that rebuilds its index lets go of the old one when the new one stands: the
        # index goes when the tensors over its tables have gone
        state["index"] = lsh.LshIndex(state["keys"])
        keys, ids = _tables(state["index"])
        return {"keys": keys, "ids": ids}
    data = state["data"]
    if kind == "dense":
        return lsh.project_e2lsh(params, data) if case["out"] == "project" else lsh.hash_e2lsh(params, data)
    if kind == "signs":
        return lsh.hash_signs(params, data)
    if kind == "mips":
        kappa2 = lsh.mips_kappa(params, data)
        return {"kappa2": kappa2, "ids": lsh.hash_mips_data(params, data, kappa2)}
    if case["out"] == "keys":
        return lsh.hash_fastlsh_keys(params, data, L)
    if case["out"] == "both":
        return lsh.hash_fastlsh_ids_keys(params, data, L)
    if case["out"] == "project":
        return lsh.project_fastlsh(params, data)
    return lsh.hash_fastlsh(params, data)


def work(case):
    """Bytes: vectors in, results out, each function's samples (a coordinate and a coefficient) or
    dense coefficients once.  Operations: two a sampled coordinate and function."""
    N, n, k, m, L = case["N"], case["n"], case["k"], case["m"], case.get("L", 1)
    kind = case["kind"]
    functions = 4 * k * m if kind == "dense" else 8 * k * m
    if kind == "index":
        return {"bytes": 8 * N * L + 12 * N * L, "flops": 0}
    if kind == "query":
        Q = case["Q"]
        seen = case["limit"] or 480  # candidates of a query, as counted
        # keys out, the two ends of every bucket out, the candidates' ids and vectors in
        return {"bytes": 4 * Q * n + functions + 16 * Q * L + Q * seen * (4 + 4 * n) + 8 * Q,
                "flops": 2 * Q * k * m + 3 * Q * seen * n}
    out = {"signs": 8 * ((k + 63) // 64), "mips": 4 * k}.get(kind) or {
        "ids": 4 * k, "project": 4 * k, "keys": 8 * L, "both": 4 * k + 8 * L}[case["out"]]
    flops = 2 * N * k * m
    if kind == "mips":  # the norms of the sampled coordinates too
        flops += 2 * N * L * m
        functions = 4 * k * m + 4 * L * m
    return {"bytes": 4 * N * n + N * out + functions, "flops": flops}


def tolerance(case):
    """Four times what the path was seen to be off from the same sums in 64 bits.  The relative error
    of m-term projections comes to 2e-8 sqrt(m) (2.0e-7 at m = 128, 4.7e-7 at 960, 1.1e-6 at 3717,
    2.3e-6 at 14174); an id differs where that error crosses the edge of a bucket, a share of 2e-8 m
    times the size of a coordinate over the width (7e-6 at the dense 960-dimensional case, 1e-4 at 3717
    dimensions of bytes), a key where one of its g ids does.  Sign words: 1.3e-4 where they are
    formed from two-term splits (n = 128).  Two values of a small result may differ in any case."""
    kind = case["kind"]
    if kind == "index":
        return "exact"
    rows, k, m, L = case["Q"] if kind == "query" else case["N"], case["k"], case["m"], case.get("L", 1)
    if kind == "signs":
        share, words = 5e-4, (k + 63) // 64
    else:
        size = {"bytes": 150.0, "unit": 0.6, "normal": 1.0}[case["dist"]]
        share, words = max(4e-6, 8e-8 * m * size / case["w"]), k
        if kind == "query" or case.get("out") in ("keys", "both"):
            share, words = share * (k // L), L
    return {"rel": 8e-8 * math.sqrt(max(m, 16)), "differ": min(0.01, share + 2 / (rows * words))}
