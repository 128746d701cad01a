"""The radix sorts at the sizes where their plan changes: pairs sorted by one workgroup (up to 4096), passes of two
launches (up to 96 tiles of 1024 or 2048 keys), passes of three, tiles with remainders; in every key and payload
width the pipeline sorts (records of one graph and of a batch, incidence entries, weights, rows, chains, graphs)."""
import numpy as np
import pytest

import synth
import test_gpu_batch as batch
import test_gpu_parity as undirected

pytestmark = pytest.mark.gpu
SIZES = [2047, 2048, 2049, 4095, 4096, 4097, 49152, 49153, 98304, 98305, 196608, 196610]


@pytest.mark.parametrize("n", SIZES)
def test_one_graph(n):
    V = max(2, n // 15)
    src, dst, t = synth.chung_lu_bursts(n, V, 4000 + n)
    undirected.assert_parity(src, dst, t, V, 5, "n=%d" % n)


@pytest.mark.parametrize("n", SIZES[:8])
def test_ranked_weights(n, monkeypatch):
    V = max(2, n // 15)
    src, dst, t = synth.chung_lu_bursts(n, V, 5000 + n)
    monkeypatch.setenv("CE_WEIGHT_RANKS", "1")
    undirected.assert_parity(src, dst, t * 1000003, V, 5, "ranked n=%d" % n)


@pytest.mark.parametrize("n", [4096, 4097, 98305])
def test_batch_of_that_many_records(n):
    cuts = np.array([0, n // 3, n // 3 + 1, n // 2, n])
    graphs = []
    for g in range(4):
        k = int(cuts[g + 1] - cuts[g])
        V = max(2, k // 15)
        graphs.append((*synth.chung_lu_bursts(k, V, 6000 + n + g), V))
    batch.check_batch_vs_oracle(graphs, 5, "n=%d" % n)
