"""Borůvka's node tree at the sizes where its plan changes: calls that one workgroup finishes alone (up to 8192
skeleton slots), calls with enqueued slots and a one-workgroup rest, list tiles with remainders, hook chains as
long as the input, one hub, isolated pairs, equal keys on parallel hyperedges; every output against the oracle."""
import numpy as np
import pytest

import synth
import test_gpu_hyper as hyper
import test_gpu_parity as undirected

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 511, 512, 513, 4095, 4096, 4097, 8193, 70001])
def test_sizes(n):
    V = max(2, n // 9)
    src, dst, t = synth.chung_lu_bursts(n, V, 900 + n)
    undirected.assert_parity(src, dst, t, V, 5, "bursts n=%d" % n)


@pytest.mark.parametrize("n", [3000, 60000])
@pytest.mark.parametrize("shape", ["growing gaps", "shrinking gaps", "hub", "pairs"])
def test_shapes(shape, n):
    i = np.arange(n, dtype=np.int64)
    src, dst = i.astype(np.int32), (i + 1).astype(np.int32)  # a path: record k meets only k - 1 and k + 1
    t = np.cumsum(i)
    if shape == "shrinking gaps":
        t = np.cumsum(n - i)
    elif shape == "hub":
        src, t = np.zeros(n, np.int32), np.random.default_rng(n).integers(0, n // 4, n)
    elif shape == "pairs":
        src, dst = (i // 2 * 2).astype(np.int32), (i // 2 * 2 + 1).astype(np.int32)
    undirected.assert_parity(src, dst, t.astype(np.int64), n + 1, 3, "%s n=%d" % (shape, n))


@pytest.mark.parametrize("n", [700, 9000])
def test_parallel_hyperedges(n):
    # every hyperedge shares all three members with its neighbours in time: each row is emitted three times
    members = np.tile(np.arange(3, dtype=np.int32), n) + 3 * np.repeat(np.arange(n, dtype=np.int32) // 50, 3)
    off = 3 * np.arange(n + 1, dtype=np.int64)
    t = np.random.default_rng(n).integers(0, n, n)
    hyper.check(members, off, t.astype(np.int64), int(members.max()) + 1, 4, "parallel n=%d" % n)
