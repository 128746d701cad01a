"""Small calls whose components only halve a round while many edges stay between them (a nested path, its records' second
vertices at random): the one workgroup that ends such calls gets a long list, which is thinned before it, from 2^18
skeleton slots on; and calls around the lines from which the list is thinned, lists are split and an asynchronous call
splits. Against the oracle; and the time of such inputs against that of as many random records."""
import time

import numpy as np
import pytest

import oracle
import test_gpu_chains as chains
import test_gpu_hyper as hyper

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def nested(n):
    k = np.arange(1, n, dtype=np.int64)
    return np.concatenate([[0], np.cumsum((k & -k) * 8 + 1)])[:n]


def one_path(n, deg, seed=1):
    G = max(1, n // deg)
    d = 1 + np.random.default_rng(seed).integers(0, G, n)
    return np.zeros(n, np.int32), d.astype(np.int32), nested(n), G + 1


def two_paths(n, deg, seed=1):
    """The gaps of the second path are larger than all edges of the first: its edges are the heavy ones of a split."""
    rng = np.random.default_rng(seed)
    h, G = n // 2, max(1, n // 2 // deg)
    s = np.repeat(np.array([0, 1], np.int32), [h, n - h])
    d = 2 + np.concatenate([rng.integers(0, G, h), G + rng.integers(0, G, n - h)])
    return s, d.astype(np.int32), np.concatenate([nested(h), nested(n - h) * 4096]), 2 * G + 2


def random_records(n, deg, seed=1):
    rng = np.random.default_rng(seed)
    V = max(2, 2 * n // deg)
    s = rng.integers(0, V - 1, n)
    return s.astype(np.int32), (s + 1).astype(np.int32), rng.integers(0, 60 * n, n), V


@pytest.mark.parametrize("shape", [one_path, two_paths])
@pytest.mark.parametrize("n, deg", [(4097, 4), (50_000, 4), (131_072, 4), (131_073, 4), (131_073, 64), (262_144, 16),
                                    (524_288, 4), (1_048_575, 4), (1_048_576, 4)])
def test_paths(shape, n, deg):
    s, d, t, V = shape(n, deg)
    chains.check(s, d, t, V, 5, "%s deg %d" % (shape.__name__, deg))


def test_parallel_hyperedges():
    n = 90_000
    rng = np.random.default_rng(3)
    m = np.stack([np.zeros(n, np.int64), 1 + rng.integers(0, 200, n), 201 + rng.integers(0, 3, n)], 1).astype(np.int32)
    hyper.check(m.reshape(-1), 3 * np.arange(n + 1, dtype=np.int64), nested(n), 204, 4, "nested, parallel")


@pytest.mark.parametrize("n, split", [(700_000, None), (1_500_000, None), (20_000, "300")])
def test_asynchronous(n, split, monkeypatch):
    import paper_2311_10337_amd as ce
    if split:
        monkeypatch.setenv("CE_SPLIT_MIN_EDGES", split)
    s, d, t, V = two_paths(n, 8)
    dev = torch.device("cuda:0")
    ins = [torch.from_numpy(x).to(dev) for x in (s, d, t)]
    outs = ce.Outputs(n, 5, dev)
    ws = torch.empty(ce.workspace_bytes(n, V, 5), dtype=torch.uint8, device=dev)
    hdr = torch.zeros(ce.hdr_words(1), dtype=torch.int64, device=dev)
    ce.cluster_edges_async(*ins, 5, V, outs, ws, hdr, time_bits=int(t.max()).bit_length())
    got = ce.to_numpy(ce.async_result(outs, n, hdr))
    ref = oracle.cluster(s, d, t, 5, V, tier=1)
    assert ref.status == 0
    for f in chains.undirected.FIELDS:
        assert np.array_equal(got[f], getattr(ref, f)), f


@pytest.mark.parametrize("shape, n", [(one_path, 500_000), (two_paths, 1_000_000), (two_paths, 2_000_000)])
def test_time(shape, n):
    import paper_2311_10337_amd as ce
    ms = {}
    for f in (random_records, shape):
        s, d, t, V = f(n, 4)
        ins = [torch.from_numpy(x).cuda() for x in (s, d, t)]
        outs = ce.Outputs(n, 5, ins[0].device)
        ws = torch.empty(ce.workspace_bytes(n, V, 5), dtype=torch.uint8, device="cuda")
        for rep in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ce.cluster_edges(*ins, 5, V, outputs=outs, workspace=ws)
            torch.cuda.synchronize()
            ms[f.__name__] = (time.perf_counter() - t0) * 1e3
    print("[gpu-rest] n=%d %s" % (n, ms), flush=True)
    assert ms[shape.__name__] < 3 * ms["random_records"]
