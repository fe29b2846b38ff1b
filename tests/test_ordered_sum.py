"""The entry rule's ordered float64 column sums.

tests/sum_harness.cpp compiles the library's run arithmetic
(csrc/ordered_sum.hpp) for the host and compares it with a plain sequential
loop, bit for bit; on the GPU the entry node must be the oracle's (a column
of neighbouring floats round the mean makes the entry name the mean itself).
"""
import subprocess
from pathlib import Path

import numpy as np
import pytest

ROOT = Path(__file__).resolve().parents[1]
KINDS = ["drift", "walk", "fall", "mixed", "ties", "whole", "flip", "zeros", "tiny", "huge", "nan", "inf"]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    exe = tmp_path_factory.mktemp("sum") / "sum_harness"
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-Wall", "-o", str(exe),
                    str(ROOT / "tests" / "sum_harness.cpp")], check=True)
    return exe


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 255, 256, 257, 5000, 300_000])
def test_runs_equal_the_plain_loop(harness, kind, n):
    for seed in range(3):
        out = subprocess.run([str(harness), kind, str(n), str(seed)], capture_output=True, text=True, check=True).stdout
        f = out.split()
        assert f[3] == "1", out
        if n == 300_000 and kind in ("drift", "walk", "fall", "whole", "flip"):
            assert int(f[1]) < 100, out   # few of the 1,172 runs are summed term by term


@pytest.mark.gpu
@pytest.mark.parametrize("n,D,kind", [(1, 1, "drift"), (256, 3, "walk"), (257, 96, "drift"), (1024, 7, "walk"), (1025, 7, "walk"),
                                      (20_000, 1, "drift"),
                                      (20_000, 1, "flip"), (30_001, 65, "walk"), (30_001, 1, "whole")])
def test_entry_is_the_oracles(n, D, kind):
    import torch
    assert torch.cuda.is_available()   # before the library: both then share one HIP runtime
    import paper_2607_04415_amd as g
    from oracle import load
    rng = np.random.default_rng(n + D)
    x = rng.standard_normal((n, D)).astype(np.float32) * np.float32(0.1)
    if kind == "drift":
        x += np.float32(0.4)
    elif kind == "whole":
        x = rng.integers(0, 256, (n, D)).astype(np.float32)
    elif kind == "flip":
        x = np.where(np.arange(n)[:, None] % 2, np.float32(-1), np.float32(1)).repeat(D, 1).astype(np.float32)
    if n > 100:
        # neighbouring floats round the mean: the nearest node names the mean
        for _ in range(3):
            mean = (np.add.accumulate(x.astype(np.float64), axis=0)[-1] / n).astype(np.float32)
            x[:33] = mean + np.spacing(mean) * np.arange(-16, 17, dtype=np.float32)[:, None]
    graph = np.full((n, 4), 0xFFFFFFFF, np.uint32)
    ix = g.Index(x, graph)
    assert ix.info["entry"] == load().medoid(x)
    ix.close()
