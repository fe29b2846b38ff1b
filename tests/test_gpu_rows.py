"""Resident search over row lengths, arrangements and placements, by a wave
per query and by a team of waves per query, against the oracle: every answer
bit, ids and distances.  Lengths are the edges of the 16-byte units and
128-byte lines that the kernels read."""
import numpy as np
import pytest

from conftest import wave_per_query_batch

pytestmark = pytest.mark.gpu

N = 700


def make(dtype, D, R, seed):
    rng = np.random.default_rng(seed)
    if dtype == "u8":
        x = rng.integers(0, 256, (N, D)).astype(np.uint8)
        q = rng.integers(0, 256, (1500, D)).astype(np.uint8)
    else:
        x = rng.standard_normal((N, D)).astype(np.float32)
        q = rng.standard_normal((1500, D)).astype(np.float32)
    graph = rng.integers(0, N, (N, R)).astype(np.uint32)
    graph[rng.random((N, R)) < 0.1] = 0xFFFFFFFF   # lists of different lengths; ids repeat too
    return x, q, graph


def check(dtype, D, R, k, L, W, layout, placed, counts=(1, 40, None)):
    """counts: batch sizes; None is one that runs a wave per query."""
    import torch
    assert torch.cuda.is_available()   # before the library: both then share one HIP runtime
    import paper_2607_04415_amd as g
    from oracle import load
    x, q, graph = make(dtype, D, R, 1000 * D + R)
    n2s = np.random.default_rng(D).permutation(N).astype(np.uint32) if placed else None
    ix = g.Index(x, graph, node_to_slot=n2s, vectors_first=layout == "vectors")
    orc = load()
    oids, od, oc, _ = orc.pack(x, graph).search(q, k, L, W, ix.info["entry"], threads=8)
    for nq in counts:
        rows = np.arange(nq or wave_per_query_batch(torch)) % len(q)
        ids, dists, st = ix.search(torch.from_numpy(q[rows]).cuda(), k, L, W)
        assert np.array_equal(ids.cpu().numpy().view(np.uint32), oids[rows]), (nq, "ids")
        assert np.array_equal(dists.cpu().numpy().view(np.uint32), od[rows].view(np.uint32)), (nq, "distances")
        assert st["expansions"] == int(oc["expansions"][rows].sum())
    ix.close()


@pytest.mark.parametrize("layout,placed", [("vectors", False), ("contiguous", False), ("vectors", True),
                                           ("contiguous", True)])
@pytest.mark.parametrize("D", [4, 32, 36, 60, 64, 100, 128, 132, 196, 256, 260, 512])
def test_u8_rows(D, layout, placed):
    check("u8", D, 20, 10, 40, 4, layout, placed)


@pytest.mark.parametrize("layout,placed", [("vectors", False), ("contiguous", False), ("contiguous", True)])
@pytest.mark.parametrize("D", [1, 3, 4, 5, 8, 9, 31, 32, 33, 64, 65, 96, 97, 128, 129, 160, 192, 223, 256])
def test_f32_rows(D, layout, placed):
    check("f32", D, 20, 10, 40, 4, layout, placed)


# frontier registers (L <= 64, 128, 256), beams of one and several groups, rows
# of up to 256 ids, a beam wider than a team
@pytest.mark.parametrize("dtype,D", [("u8", 128), ("u8", 100), ("f32", 96), ("f32", 160)])
@pytest.mark.parametrize("R,k,L,W", [(64, 10, 64, 1), (64, 64, 64, 9), (65, 10, 65, 8), (1, 1, 128, 128), (96, 100, 128, 5),
                                     (256, 10, 129, 3), (33, 200, 256, 256), (12, 12, 12, 12),
                                     # each width of a team with each frontier: up to 128, 256 and more ids
                                     (128, 10, 100, 1), (43, 10, 200, 3), (129, 10, 100, 1), (64, 10, 200, 4),
                                     (16, 20, 200, 1), (86, 10, 64, 3), (43, 10, 64, 3)])
def test_beams(dtype, D, R, k, L, W):
    check(dtype, D, R, k, L, W, "vectors", False, counts=(3, 512, None))


# a wave per query with each number of frontier registers: beams of two groups,
# groups of up to four batches of 64, placed and not
@pytest.mark.parametrize("layout,placed", [("vectors", False), ("vectors", True), ("contiguous", True)])
@pytest.mark.parametrize("L", [64, 100, 200])
@pytest.mark.parametrize("dtype,D", [("u8", 16), ("u8", 64), ("u8", 128), ("u8", 200), ("u8", 300), ("f32", 5),
                                     ("f32", 20), ("f32", 32), ("f32", 64), ("f32", 90), ("f32", 96), ("f32", 128),
                                     ("f32", 150), ("f32", 256)])
def test_wave_per_query(dtype, D, L, layout, placed):
    # 1,000: past the teams of eight, at most one wave per SIMD
    check(dtype, D, 64, 50, L, 8, layout, placed, counts=(1000, None))
