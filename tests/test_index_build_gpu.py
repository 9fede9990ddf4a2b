"""Building an index: the tables are the stable sort of every column of keys, whatever the memory
they are built in was used for before."""
import ctypes
import os
import subprocess
import sys
import threading

import numpy as np
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


class _View:
    def __init__(self, address, shape, kind):
        self.__cuda_array_interface__ = {"data": (address, False), "shape": shape, "typestr": kind, "version": 2}


def _tables(lsh, ix):
    """Copies of the sorted keys [L, N] (signed views of the unsigned keys) and the ids."""
    keys, ids = ctypes.c_void_p(), ctypes.c_void_p()
    assert lsh.load_library().lsh_index_tables(ix.handle, None, None, ctypes.byref(keys), ctypes.byref(ids)) == 0
    shape = (ix.L, ix.N)
    return (torch.as_tensor(_View(keys.value, shape, "<i8"), device="cuda").clone(),
            torch.as_tensor(_View(ids.value, shape, "<i4"), device="cuda").clone())


def _check(lsh, ix, keys, label):
    got_keys, got_ids = _tables(lsh, ix)
    # unsigned order: flip the sign bit, sort as signed numbers
    flipped = keys.t().contiguous() ^ torch.tensor(-2 ** 63, device="cuda")
    want, order = torch.sort(flipped, dim=1, stable=True)
    assert torch.equal(got_keys, want ^ torch.tensor(-2 ** 63, device="cuda")), label
    assert torch.equal(got_ids.long(), order), label


def _random_keys(N, L, distinct, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pool = torch.randint(-2 ** 63, 2 ** 63 - 1, (distinct, L), generator=g, device="cuda")
    return torch.gather(pool, 0, torch.randint(0, distinct, (N, L), generator=g, device="cuda"))


def _keys_of(kind, N, L, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    some = lambda *shape: torch.randint(-2 ** 63, 2 ** 63 - 1, shape, generator=g, device="cuda")
    below = lambda k: torch.randint(0, k, (N, L), generator=g, device="cuda")
    if kind == "random":
        return some(N, L)
    if kind == "one":
        return torch.full((N, L), -5, device="cuda")
    if kind == "half":          # one key half of the time
        return torch.where(below(2) == 0, some(N, L), torch.full((N, L), 77, device="cuda"))
    if kind == "few":           # the keys of tables of one function: ids, negative ones as 32 unsigned bits
        return (below(20) - 10) & 0xFFFFFFFF
    if kind == "groups":        # keys that agree in all functions but the last
        return some(max(1, N // 40), L)[below(max(1, N // 40)), torch.arange(L, device="cuda")] + ((below(5) - 2) & 0xFFFFFFFF)
    if kind == "ends":
        return torch.tensor([0, -1, -2, 2 ** 63 - 1, -2 ** 63], device="cuda")[below(5)]
    return (torch.arange(N, device="cuda")[:, None] * 3 + torch.arange(L, device="cuda")) * (1 if kind == "rising" else -1)


# around a tile of 4096 rows, buckets of one workgroup's 4096 and 8192 pairs, four tables at a time, and the line between
# the two sorts at 2^20
@pytest.mark.parametrize("kind", ["random", "one", "half", "few", "groups", "ends", "rising", "falling"])
@pytest.mark.parametrize("N,L", [(1, 1), (2, 5), (4095, 2), (4096, 3), (4097, 4), (8193, 1), (70001, 6), (300000, 1),
                                 (2 ** 20, 1), (2 ** 20 + 1, 1)])
def test_tables_of_all_kinds_of_keys(lsh, kind, N, L):
    print(f"{kind} N={N} L={L}", flush=True)
    keys = _keys_of(kind, N, L, N + L).contiguous()
    with lsh.LshIndex(keys) as ix:
        _check(lsh, ix, keys, f"{kind} N={N} L={L}")


def _sampled_rows(N, L):
    """The rows by whose keys the buckets are divided (index_sort.hip: plan_of, sort_splitters)."""
    buckets = 1
    while buckets * 2048 < N:
        buckets *= 2
    while buckets < 512 and buckets * L < 512 and buckets * 512 <= N:
        buckets *= 2
    j = np.arange(16 * buckets, dtype=np.uint64)
    first, end = j * N // len(j), (j + 1) * N // len(j)
    mixed = ((j * 0x9E3779B1 ^ 0x85EBCA6B) & 0xFFFFFFFF) * 0xC2B2AE35 & 0xFFFFFFFF
    return torch.as_tensor((first + ((mixed ^ mixed >> np.uint64(15)) * (end - first) >> np.uint64(32))).astype(np.int64), device="cuda")


# Keys of which the sample shows nothing: it meets key 0 only, and all others lie in the last bucket.  Some 6000 of them are
# sorted by one workgroup of 1024 threads; more part by part: keys of all sizes, a key that alone is more than a
# part, and a cluster a few thousand wide among some that are far off.  (300000 and 2^20 rows: 512 buckets, as many as there can be.)
@pytest.mark.parametrize("N,L", [(20000, 3), (70001, 1), (300000, 1)])
@pytest.mark.parametrize("kind", ["some", "all", "heavy", "cluster"])
def test_tables_of_keys_that_the_sample_misses(lsh, kind, N, L):
    print(f"{kind} N={N} L={L}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    keys = torch.randint(-2 ** 63, 2 ** 63 - 1, (N, L), generator=g, device="cuda")
    below = lambda k: torch.randint(0, k, (N, L), generator=g, device="cuda")
    if kind == "some":
        keys[below(N) >= 6000] = 0
    elif kind == "heavy":
        keys[below(2) == 0] = -77
    elif kind == "cluster":
        keys = torch.where(below(1000) == 0, keys, 0x5EED5EED5EED5EED + below(5000))
    keys[_sampled_rows(N, L)] = 0
    with lsh.LshIndex(keys) as ix:
        _check(lsh, ix, keys, f"{kind} N={N} L={L}")


def test_largest_table_of_keys_that_the_sample_misses(lsh):
    N = 2 ** 20
    keys = torch.arange(N, device="cuda")[:, None] // 3 * 0x9E3779B9
    keys[_sampled_rows(N, 1)] = 0
    with lsh.LshIndex(keys.contiguous()) as ix:
        _check(lsh, ix, keys, "2^20")


def test_keys_on_no_boundary_of_16_bytes(lsh):
    keys = _random_keys(9001, 2, 4000, 3)
    moved = torch.empty(keys.numel() + 1, dtype=torch.int64, device="cuda")[1:].view(9001, 2)
    moved.copy_(keys)
    assert moved.data_ptr() % 16 == 8
    with lsh.LshIndex(moved) as ix:
        _check(lsh, ix, keys, "keys at 8 modulo 16")


def test_tables_built_in_memory_of_earlier_indexes(lsh):
    """Indexes of several sizes built, used and dropped in turn: each must be whole while others come
    and go in the memory that earlier ones and their scratch left behind."""
    alive = []
    for i, (N, L) in enumerate([(5000, 3), (70000, 4), (5000, 3), (300, 40), (70000, 4), (68000, 4), (1, 1), (90000, 2)]):
        print(f"index {i}: N={N} L={L}", flush=True)
        keys = _random_keys(N, L, max(1, N // 3), i)
        alive.append((lsh.LshIndex(keys), keys))
        if len(alive) == 3:
            alive.pop(0)[0].close()
        for ix, k in alive:
            _check(lsh, ix, k, f"index {i}")
    for ix, _ in alive:
        ix.close()


def test_indexes_built_by_several_threads_and_streams(lsh):
    sizes = [(40000, 4), (40000, 4), (36000, 4), (9000, 7)]
    keys = [_random_keys(N, L, N // 2, 50 + i) for i, (N, L) in enumerate(sizes)]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(6):
                    with lsh.LshIndex(keys[i]) as ix:
                        _check(lsh, ix, keys[i], f"thread {i}")
        except BaseException as e:      # noqa: BLE001 -- reported by the main thread
            bad.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


_CAPTURE = """
import torch
import paper_2309_15479_amd as lsh
keys = torch.randint(0, 5000, (20000, 3), device="cuda")
other = lsh.LshIndex(keys)
lsh.LshIndex(keys).close()
torch.cuda.synchronize()
try:
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        try:
            built = lsh.LshIndex(keys)
            print("built", flush=True)
        except lsh.LshError:
            print("refused", flush=True)
except RuntimeError:
    pass
"""


def test_destroying_an_index_waits_for_work_on_any_stream(lsh):
    """Another stream may still read the tables: their memory is used again only after that."""
    keys = _random_keys(20000, 3, 5000, 9)
    indexes = [lsh.LshIndex(keys), lsh.LshIndex(keys)]
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    big = torch.randn((4096, 4096), device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(100):
            big = big @ big * 1e-2
        done.record()
    assert not done.query()
    indexes.pop().close()
    assert done.query()
    indexes.pop().close()


_DESTROY_IN_CAPTURE = """
import threading
import torch
import paper_2309_15479_amd as lsh
keys = torch.randint(0, 5000, (20000, 3), device="cuda")
indexes = [lsh.LshIndex(keys) for _ in range(3)]
data = torch.randn((1000, 128), device="cuda")
out = torch.empty((1000, 64), dtype=torch.int32, device="cuda")
with lsh.LshParams(128, 64, 32, 4.0, 1) as p:
    want = lsh.hash_fastlsh(p, data, out=out).clone()
    torch.cuda.synchronize()
    for mode in ("relaxed", "thread_local"):
        ix = indexes.pop()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode=mode):
            lsh.hash_fastlsh(p, data, out=out)
            if mode == "relaxed":
                ix.close()
            else:
                other = threading.Thread(target=ix.close)
                other.start()
                other.join()
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        print(mode, "captured", flush=True)
"""


def test_destroying_an_index_leaves_a_capture_alone(lsh):
    """As freeing memory does: in the capturing thread in relaxed mode, in another one in the others."""
    r = subprocess.run([sys.executable, "-c", _DESTROY_IN_CAPTURE], capture_output=True, text=True, timeout=100,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert "relaxed captured" in r.stdout and "thread_local captured" in r.stdout, r.stdout + r.stderr


def test_build_is_refused_under_capture(lsh):
    """Memory that earlier builds left must not make a capture take what it may not hold (in a process
    of its own: the refused call invalidates the capture and what the stream does after it)."""
    r = subprocess.run([sys.executable, "-c", _CAPTURE], capture_output=True, text=True, timeout=100,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert "refused" in r.stdout and "built" not in r.stdout, r.stdout + r.stderr
