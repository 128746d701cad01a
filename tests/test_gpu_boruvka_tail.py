"""Calls whose enqueued Boruvka slots end before the forest does, so that one workgroup finishes them: in plain rounds,
among the light edges of a split, with its heavy edges still parked; on inputs whose components only halve a round
(a path of records with nested gaps). Every output against the oracle."""
import numpy as np
import pytest

import synth
import test_gpu_hyper as hyper
import test_gpu_parity as undirected

pytestmark = pytest.mark.gpu


def nested_path(bits):
    """Records along a path of vertices; the gap before record k is larger the more zero bits k ends with, so pairs
    merge first, then pairs of pairs: as many rounds as bits."""
    n = 1 << bits
    k = np.arange(1, n, dtype=np.int64)
    t = np.concatenate([[0], np.cumsum((k & -k) * 8 + 1)])
    i = np.arange(n, dtype=np.int32)
    return i, i + 1, t, n + 1


@pytest.mark.parametrize("split", [0, 64, 1024, 1 << 20])
@pytest.mark.parametrize("bits", [6, 11, 13, 16])
def test_halving(bits, split, monkeypatch):
    monkeypatch.setenv("CE_SPLIT_MIN_EDGES", str(split))
    undirected.assert_parity(*nested_path(bits), 3, "nested path 2^%d, split %d" % (bits, split))


@pytest.mark.parametrize("thr", [2, 8, 64, 512])
@pytest.mark.parametrize("n", [40, 300, 5000, 60001])
def test_split_and_rest(n, thr, monkeypatch):
    monkeypatch.setenv("CE_SPLIT_MIN_EDGES", str(thr))
    V = max(2, n // 40)
    src, dst, t = synth.chung_lu_bursts(n, V, 300 + n + thr)
    undirected.assert_parity(src, dst, t, V, 4, "n=%d thr=%d" % (n, thr))


@pytest.mark.parametrize("thr", [2, 64])
def test_split_of_parallel_hyperedges(thr, monkeypatch):
    monkeypatch.setenv("CE_SPLIT_MIN_EDGES", str(thr))
    n = 900
    members = np.tile(np.arange(3, dtype=np.int32), n) + 3 * np.repeat(np.arange(n, dtype=np.int32) // 50, 3)
    off = 3 * np.arange(n + 1, dtype=np.int64)
    t = np.random.default_rng(n).integers(0, n, n)
    hyper.check(members, off, t.astype(np.int64), int(members.max()) + 1, 4, "parallel, split %d" % thr)


@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1])
def test_around_the_line(n):
    V = n // 30
    src, dst, t = synth.chung_lu_bursts(n, V, n)
    undirected.assert_parity(src, dst, t, V, 5, "n=%d" % n)


@pytest.mark.parametrize("split", [0, 1 << 20])
def test_many_rounds_past_the_line(split, monkeypatch):
    # 22 rounds: a synchronous call looks for the end after 12 slots and every 4 from there
    monkeypatch.setenv("CE_SPLIT_MIN_EDGES", str(split))
    undirected.assert_parity(*nested_path(22), 3, "nested path 2^22, split %d" % split)
