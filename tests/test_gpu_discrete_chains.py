"""Calls with thresholds whose level tops lie at the end of one long chain: records of one vertex at regular or growing
intervals, all forest rows in one level (or a level of its own for the last), at the record counts around which another
round of pointer jumping is needed; single calls (repeated: in-place updates may or may not help a round), a batch, a
captured call; every output against the oracle."""
import numpy as np
import pytest

import test_gpu_discrete as discrete

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def hub(n, shape):
    k = np.arange(n, dtype=np.int64)
    return (np.zeros(n, np.int32), np.arange(1, n + 1, dtype=np.int32), 60 * k if shape == "regular" else np.cumsum(k),
            n + 1)


@pytest.mark.parametrize("n", [2, 6, 7, 22, 102, 502, 503, 504, 511, 512, 513, 2502, 2503, 12502, 12503, 62502, 62503,
                               65535, 65536, 65537, 312503])
@pytest.mark.parametrize("shape", ["regular", "growing"])
def test_one_level(n, shape):
    ce = discrete._ce()
    s, d, t, V = hub(n, shape)
    top = int(t[-1] - t[-2])
    for thr in ([top], [0, top - 1, top] if top > 1 else [0, top]):
        ref = discrete.ref_dict(s, d, t, V, 5, thr)
        for rep in range(8 if n <= 600 else 3):
            got = ce.to_numpy(ce.cluster_edges(*discrete.dev_arrays(s, d, t), 5, V, thresholds=thr))
            discrete.same(got, ref, "%s n=%d thr=%s" % (shape, n, thr))


def test_batch():
    ce = discrete._ce()
    graphs = [hub(n, "regular") for n in (1, 510, 1)]  # 511 rows at most, and a chain of 509
    cat = lambda k, dt: np.concatenate([np.asarray(g[k], dt) for g in graphs])
    eoff = np.cumsum([0] + [len(g[0]) for g in graphs]).astype(np.int64)
    voff = np.cumsum([0] + [g[3] for g in graphs]).astype(np.int64)
    ins = discrete.dev_arrays(cat(0, np.int32), cat(1, np.int32), cat(2, np.int64))
    for rep in range(8):
        br = ce.cluster_batch(*ins, eoff, voff, 4, thresholds=[60])
        for g, (s, d, t, V) in enumerate(graphs):
            discrete.same(br.graph(g), discrete.ref_dict(s, d, t, V, 4, [60]), "batch graph %d" % g)


@pytest.mark.parametrize("n", [512, 65536])
def test_captured(n):
    ce = discrete._ce()
    s, d, t, V = hub(n, "regular")
    ins = discrete.dev_arrays(s, d, t)
    dev = ins[0].device
    outs = ce.Outputs(n, 5, dev)
    ws = torch.empty(ce.workspace_bytes(n, V, 5, thresholds=[60]), dtype=torch.uint8, device=dev)
    hdr = torch.zeros(ce.hdr_words(1), dtype=torch.int64, device=dev)
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream(device=dev)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            ce.cluster_edges_async(*ins, 5, V, outs, ws, hdr, time_bits=24, stream=torch.cuda.current_stream(),
                                   thresholds=[60])
    torch.cuda.synchronize()
    ref = discrete.ref_dict(s, d, t, V, 5, [60])
    for rep in range(5):
        outs.t["dd_top"].fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        got = ce.to_numpy(ce.async_result(outs, n, hdr))
        for f in ("dd_level", "dd_top"):
            got[f] = outs.t[f][:got["m"]].cpu().numpy()
        discrete.same(got, ref, "replay %d" % rep)
