"""The dendrogram read off the Borůvka tree, where its plan and its chains change: calls whose levels one workgroup
sums and calls with enqueued levels, chains longer than a wave's stretch (hubs, one growing path), forests cut by
max_dt down to a few rows or none, a filter split inside the tree; every output against the oracle."""
import os

import numpy as np
import pytest

import oracle
import synth
import test_gpu_parity as undirected

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(src, dst, t, V, M, label, max_dt=-1):
    import paper_2311_10337_amd as ce
    print("[gpu-chains] %s n=%d max_dt=%d" % (label, len(t), max_dt), flush=True)
    ref = oracle.cluster(src, dst, t, M, V, tier=1, max_dt=max_dt)
    assert ref.status == 0
    dev = torch.device("cuda:0")
    ins = [torch.from_numpy(np.ascontiguousarray(x, k)).to(dev) for x, k in ((src, np.int32), (dst, np.int32),
                                                                             (t, np.int64))]
    got = ce.to_numpy(ce.cluster_edges(*ins, M, V, max_dt=max_dt))
    assert (got["m"], got["n_clusters"], got["n_labels"]) == (ref.m, ref.n_clusters, ref.n_labels), label
    for f in undirected.FIELDS:
        assert np.array_equal(got[f], getattr(ref, f)), (label, f)


@pytest.mark.parametrize("n", [2, 5, 4096, 4097, 40000])
@pytest.mark.parametrize("max_dt", [-1, 0, 1, 50])
def test_cut_forests(n, max_dt):
    V = max(2, n // 12)
    src, dst, t = synth.chung_lu_bursts(n, V, 77 + n)
    check(src, dst, t, V, 4, "bursts", max_dt)


@pytest.mark.parametrize("n", [1025, 4096, 30000])
@pytest.mark.parametrize("shape", ["hub", "growing", "two hubs", "equal times"])
def test_long_chains(shape, n):
    rng = np.random.default_rng(n)
    src, dst = np.zeros(n, np.int32), np.arange(1, n + 1, dtype=np.int32)
    t = np.cumsum(np.arange(n, dtype=np.int64)) if shape == "growing" else rng.integers(0, 50 * n, n)
    if shape == "two hubs":
        src = (np.arange(n) % 2 * (n + 1)).astype(np.int32)
        dst[n // 2] = n + 1 if src[n // 2] == 0 else 0
    if shape == "equal times":
        t = rng.integers(0, 5, n)
    check(src, dst, t.astype(np.int64), n + 2, 3, shape)


@pytest.mark.parametrize("split", [1, 3000])
@pytest.mark.parametrize("max_dt", [-1, 120])
def test_split_inside_the_tree(split, max_dt):
    old = os.environ.get("CE_SPLIT_MIN_EDGES")
    os.environ["CE_SPLIT_MIN_EDGES"] = str(split)
    try:
        for seed in (1, 2, 3):
            src, dst, t = synth.rmat_hawkes(20000, 9, seed)
            check(src, dst, t, 1 << 9, 5, "split at %d seed %d" % (split, seed), max_dt)
    finally:
        if old is None:
            del os.environ["CE_SPLIT_MIN_EDGES"]
        else:
            os.environ["CE_SPLIT_MIN_EDGES"] = old
