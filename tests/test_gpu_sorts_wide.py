"""The radix sorts around 2^19 keys, where tiles grow from 2048 keys (256 threads) to 4096 (512 threads): one below, at
and above the line, and one key past a whole number of the wide tiles; for records (times of up to and over 32 bits),
incidence entries, rows, chains and ranked weights, and for a batch."""
import numpy as np
import pytest

import synth
import test_gpu_batch as batch
import test_gpu_parity as undirected

pytestmark = pytest.mark.gpu
LINE = 1 << 19
SIZES = [LINE // 2, LINE // 2 + 1, LINE - 1, LINE, LINE + 1, LINE + 4097]


@pytest.mark.parametrize("n", SIZES)
def test_one_graph(n):
    V = n // 15
    src, dst, t = synth.chung_lu_bursts(n, V, 7000 + n)
    undirected.assert_parity(src, dst, t, V, 5, "n=%d" % n)


@pytest.mark.parametrize("n", [LINE // 2 + 1, LINE + 4097])
def test_wide_times_and_ranked_weights(n, monkeypatch):
    V = n // 15
    src, dst, t = synth.chung_lu_bursts(n, V, 8000 + n)
    monkeypatch.setenv("CE_WEIGHT_RANKS", "1")
    undirected.assert_parity(src, dst, t * 1000003, V, 5, "ranked n=%d" % n)


def test_batch():
    n = LINE + 4097
    graphs = []
    for k in (n // 3, 1, n - n // 3 - 1):
        V = max(2, k // 15)
        graphs.append((*synth.chung_lu_bursts(k, V, 9000 + k), V))
    batch.check_batch_vs_oracle(graphs, 5, "n=%d" % n)
