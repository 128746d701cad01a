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


def light_and_heavy(n, shape):
    """Pairs of records, two halves: the first at regular gaps, smaller than any of the second, with second vertices in a
    few classes, so that a split takes its edges alone; the second half is one chain among the heavy edges."""
    h = n // 2
    k = torch.arange(h, dtype=torch.int64, device="cuda")
    j = torch.arange(h // 2, dtype=torch.int64, device="cuda")
    gaps = 11000 + (j if shape == "growing" else h // 2 - j)
    tb = (torch.cumsum(gaps, 0) - gaps)[:, None] + torch.tensor([0, 1000], device="cuda")
    t = torch.cat([10 * (k // 2) + k % 2, 10 * h + 1000000 + tb.reshape(-1)])
    cl = k // 2 % 3 * 2 + k % 2
    src = torch.zeros(2 * h, dtype=torch.int32, device="cuda")
    src[h:] = 1
    return src, torch.cat([2 + cl, 8 + cl]).int(), t, 14


@pytest.mark.parametrize("shape", ["growing", "shrinking"])
@pytest.mark.parametrize("grid, split", [(256, 1000), (256, 50000), (4096, 1000)])
def test_chain_among_heavy_edges(grid, split, shape, monkeypatch):
    monkeypatch.setenv("CE_LIST_GRID", str(grid))
    monkeypatch.setenv("CE_SPLIT_MIN_EDGES", str(split))
    s, d, t, V = light_and_heavy(300_000, shape)
    chains.check(s.cpu().numpy(), d.cpu().numpy(), t.cpu().numpy(), V, 3, "light and heavy, " + shape)


def test_time_of_a_chain_among_heavy_edges():
    import paper_2311_10337_amd as ce
    n = 16_000_000
    outs = ce.Outputs(n, 5, torch.device("cuda:0"))
    ws = torch.empty(ce.workspace_bytes(n, 14, 5), dtype=torch.uint8, device="cuda")
    ms = {}
    for shape in ("growing", "shrinking"):
        s, d, t, V = light_and_heavy(n, shape)
        for rep in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ce.cluster_edges(s, d, t, 5, V, outputs=outs, workspace=ws)
            torch.cuda.synchronize()
            ms[shape] = (time.perf_counter() - t0) * 1e3
    print("[gpu-regular] light and heavy %s" % ms, flush=True)
    assert ms["shrinking"] < 2 * ms["growing"]
