"""Records at regular, growing and shrinking intervals (and in pairs at regular intervals), in time order: every round's
hooks are one chain through all records. At the edges of a tile of nodes and where the links of all tiles get a launch
of their own, against the oracle; at sizes whose tiles are not in flight together, against the time that the same number
of records takes at random times (a walk through tiles that have not been started takes hundreds of times as long)."""
import time

import numpy as np
import pytest

import test_gpu_chains as chains

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = ("regular", "growing", "shrinking", "pairs")


def times(n, shape):
    k = np.arange(n, dtype=np.int64)
    if shape == "random":
        return np.sort(np.random.default_rng(n).integers(0, 60 * n, n))
    return {"regular": lambda: 60 * k, "growing": lambda: np.cumsum(k), "shrinking": lambda: np.cumsum(k[::-1]),
            "pairs": lambda: 60 * (k // 2) + k % 2}[shape]()


@pytest.mark.parametrize("n", [63, 513, 4095, 4096, 4097, 8200, 262143, 262145, (1 << 21) + 5])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_vertex(shape, n):
    chains.check(np.zeros(n, np.int32), np.arange(1, n + 1, dtype=np.int32), times(n, shape), n + 1, 3, shape)


@pytest.mark.parametrize("grid", [256, 1024])
@pytest.mark.parametrize("shape", SHAPES)
def test_few_workgroups(shape, grid, monkeypatch):
    monkeypatch.setenv("CE_LIST_GRID", str(grid))
    n = 300_001
    chains.check(np.arange(n, dtype=np.int32), np.arange(1, n + 1, dtype=np.int32), times(n, shape), n + 1, 3, shape)


@pytest.mark.parametrize("n", [4_000_000, 8_000_000])
def test_time_of_a_chain(n):
    import paper_2311_10337_amd as ce
    src = torch.zeros(n, dtype=torch.int32, device="cuda")
    dst = torch.arange(1, n + 1, dtype=torch.int32, device="cuda")
    outs = ce.Outputs(n, 5, src.device)
    ws = torch.empty(ce.workspace_bytes(n, n + 1, 5), dtype=torch.uint8, device="cuda")
    ms = {}
    for shape in ("random",) + SHAPES:
        t = torch.from_numpy(np.ascontiguousarray(times(n, shape))).cuda()
        for rep in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ce.cluster_edges(src, dst, t, 5, n + 1, outputs=outs, workspace=ws)
            torch.cuda.synchronize()
            ms[shape] = (time.perf_counter() - t0) * 1e3
        print("[gpu-regular] n=%d %s %.2f ms" % (n, shape, ms[shape]), flush=True)
        assert ms[shape] < 10 * ms["random"], shape
