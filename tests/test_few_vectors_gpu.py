"""Launches of few vectors deal a tile's functions (and sub-tiles) to more workgroups than launches of
many do, out of the same lists: a vector's results are the same numbers either way."""
import os
import subprocess
import sys

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


@pytest.mark.parametrize("n,k,m,L,w", [
    (4096, 2048, 64, 128, 8.0),    # lists by coordinate ranges: four functions a lane
    (4100, 1500, 40, 375, 3.0),    # three, idle lanes in the last set
    (2100, 1024, 100, 64, 4.0),    # two, and blocks of two quads
    (2500, 4000, 70, 250, 4.0),    # two workgroups along the functions already
    (4096, 512, 64, 32, 8.0),      # one: nothing to deal out
    (2101, 512, 48, 32, 4.0),      # sixteen stages for nine ranges, the last list block opening one; odd n
    (2196, 896, 71, 56, 4.0),      # the same, two functions a lane
    (8200, 640, 100, 80, 4.0),     # forty stages: four whole vectors just fit LDS
    (10240, 512, 33, 16, 4.0),     # forty ranges in them
    (10500, 600, 70, 75, 4.0),     # forty-eight: they do not
    (8200, 320, 100, 40, 4.0),     # less than 512 functions: no lists by ranges, tiles of one sub-tile
    (10500, 200, 70, 25, 4.0),
    (960, 1024, 128, 64, 1.0),     # whole-vector tiles of eight sub-tiles
    (403, 250, 100, 125, 0.75),    # the same, nothing a multiple of anything
    (1500, 700, 100, 175, 2.0),    # tiles of four sub-tiles
    (2500, 300, 100, 75, 2.0),     # tiles of two sub-tiles: the functions alone
])
def test_few_vectors_equal_many(lsh, n, k, m, L, w):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + k)
    N = 9000                       # more tiles than the chip has CUs, in every one of these shapes
    data = torch.randn((N, n), generator=g, device="cuda")
    with lsh.LshParams(n, k, m, w, 5) as p:
        many = {"ids": lsh.hash_fastlsh(p, data), "proj": lsh.project_fastlsh(p, data), "signs": lsh.hash_signs(p, data)}
        gs = k // L
        if gs & (gs - 1) == 0:
            many["keys"] = lsh.hash_fastlsh_keys(p, data, L)
        for first, count in ((0, 1), (33, 17), (5, 100), (8000, 1000), (100, 2500)):
            print(f"few vectors: n={n} k={k} m={m} first={first} count={count}", flush=True)
            part = data[first:first + count].clone()
            rows = slice(first, first + count)
            assert torch.equal(lsh.hash_fastlsh(p, part), many["ids"][rows])
            assert torch.equal(lsh.project_fastlsh(p, part), many["proj"][rows])
            assert torch.equal(lsh.hash_signs(p, part), many["signs"][rows])
            if "keys" in many:
                assert torch.equal(lsh.hash_fastlsh_keys(p, part, L), many["keys"][rows])
                ids, keys = lsh.hash_fastlsh_ids_keys(p, part, L)
                assert torch.equal(ids, many["ids"][rows]) and torch.equal(keys, many["keys"][rows])


@pytest.mark.parametrize("k,m,L,w", [(32, 30, 8, 4.0), (64, 128, 8, 3.0), (96, 32, 6, 2.0), (160, 32, 5, 0.7), (512, 32, 32, 512.0)])
def test_few_vectors_of_128_dimensions_equal_many(lsh, k, m, L, w):
    """A block of 32 functions x 32 vectors a wave: the bits of whole tiles, whose products of zero terms are skipped."""
    g = torch.Generator(device="cuda")
    g.manual_seed(k)
    N = 40000                      # beyond 1024 such blocks (2048 from 512 functions on)
    data = torch.randn((N, 128), generator=g, device="cuda")
    data[N // 2:] = (data[N // 2:] * 40).round()
    with lsh.LshParams(128, k, m, w, 5) as p:
        many = {"ids": lsh.hash_fastlsh(p, data), "proj": lsh.project_fastlsh(p, data), "signs": lsh.hash_signs(p, data),
                "keys": lsh.hash_fastlsh_keys(p, data, L)}
        for first, count in ((0, 1), (7, 31), (20000, 33), (19990, 64), (100, 1001), (23000, 2048)):
            print(f"few vectors of 128: k={k} m={m} first={first} count={count}", flush=True)
            part = data[first:first + count].clone()
            rows = slice(first, first + count)
            assert torch.equal(lsh.hash_fastlsh(p, part), many["ids"][rows])
            assert torch.equal(lsh.project_fastlsh(p, part), many["proj"][rows])
            assert torch.equal(lsh.hash_signs(p, part), many["signs"][rows])
            assert torch.equal(lsh.hash_fastlsh_keys(p, part, L), many["keys"][rows])
            ids, keys = lsh.hash_fastlsh_ids_keys(p, part, L)
            assert torch.equal(ids, many["ids"][rows]) and torch.equal(keys, many["keys"][rows])
            if m == 128:
                assert torch.equal(lsh.hash_e2lsh(p, part), lsh.hash_e2lsh(p, data)[rows])


_CAPTURED = """
import sys
import torch
import paper_2309_15479_amd as lsh
n, k, m = (int(x) for x in sys.argv[1:])
g = torch.Generator(device="cuda")
g.manual_seed(m)
data = torch.randn((9000, n), generator=g, device="cuda")
call = lsh.hash_e2lsh if m == n else lsh.hash_fastlsh
with lsh.LshParams(n, k, m, 4.0, 21) as p:
    out = torch.empty((9000, k), dtype=torch.int32, device="cuda")
    call(p, data[:8].clone())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(p, data, out=out)
    want = call(p, data)
    for _ in range(3):
        out.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    print("captured", flush=True)
"""


@pytest.mark.parametrize("n,k,m", [(960, 1024, 960), (4096, 2048, 64), (960, 1024, 128)])
def test_many_captured_after_few(lsh, n, k, m):
    """A program that has only hashed few vectors so far may capture a launch of many: another kernel, on
    first use, whose limits are raised inside the capture (they are raised once a process, hence a fresh one)."""
    r = subprocess.run([sys.executable, "-c", _CAPTURED, str(n), str(k), str(m)], capture_output=True, text=True, timeout=100,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0 and "captured" in r.stdout, r.stdout + r.stderr
