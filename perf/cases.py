"""Workloads that say how fast the framework is in use.

Every case is one call (or one burst of requests) through the package's public entry points, on seeded synthetic
inputs drawn on the GPU with the value ranges and skews of the repository's own workloads: Chung-Lu endpoints
(exponent 2.1) with Poisson-burst times, R-MAT endpoints (0.57, 0.19, 0.19, 0.05) with self-exciting per-pair times
and planted hubs, multi-recipient messages as hyperedges. Sizes run from one 500-record graph to 2e8 records, and
from 2 to 1024 graphs a batch.

All outputs are whole numbers (forest rows, tree nodes, 128-bit sums in two words, labels): they are compared for
equality, and nothing in them is rounded.
"""
import math

import numpy as np
import torch

import paper_2311_10337_amd as ce

DAY = 86400
PAPER_THRESHOLDS = [1 << i for i in range(29)]  # 2^0 .. 2^28 seconds


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # The smallest request of a serving stream, by the plain call (workspace made by the library): all latency and
        # launches.
        {"name": "request-1k", "kind": "edges", "graph": "rmat", "n": 1000, "scale": 6, "days": 90, "M": 10, "hub": 0,
         "max_dt": -1, "kept": False},
        # The median request of the serving stream, an odd size, with the workspace kept from call to call.
        {"name": "request-71k", "kind": "edges", "graph": "rmat", "n": 70711, "scale": 13, "days": 90, "M": 10,
         "hub": 0, "max_dt": -1, "kept": True},
        # The same order of size captured once as a HIP graph and replayed: a loop that enqueues and reads nothing back.
        {"name": "replay-57k", "kind": "replay", "graph": "bursts", "n": 57000, "V": 2850, "days": 30, "M": 5},
        # The repository's tiny workload: 200k records of bursty conversations over 10k people.
        {"name": "tiny-200k", "kind": "edges", "graph": "bursts", "n": 200000, "V": 10000, "days": 30, "M": 5, "hub": 0,
         "max_dt": -1, "kept": False},
        # Microsecond time stamps over a year: the weights do not fit the key and go by their ranks.
        {"name": "micros-1m", "kind": "edges", "graph": "micros", "n": 1000003, "V": 50000, "days": 365, "M": 5,
         "hub": 0, "max_dt": -1, "kept": True},
        # A thousand tenants' or time windows' graphs of very uneven size in one call.
        {"name": "batch-1024", "kind": "batch", "G": 1024, "median": 20000, "sigma": 1.5, "lo": 500, "hi": 2000000,
         "M": 5, "causal": False},
        # A burst of mixed requests through the server, from host memory to polled results.
        {"name": "serve-48", "kind": "serve", "requests": 48, "median": 70711, "sigma": 1.42, "lo": 1000,
         "hi": 2000000, "M": 10},
        # The line graph and dendrogram of the paper's own experiments: causal, 29 thresholds.
        {"name": "causal-levels-8m", "kind": "causal", "n": 8000000, "scale": 18, "days": 90, "M": 10,
         "thresholds": 29},
        # Multi-recipient messages (about 4.4 members each).
        {"name": "hyper-4m", "kind": "hyper", "n": 4000000, "V": 262144, "days": 90, "M": 10},
        # Partitions at 29 thresholds from a forest that an earlier call returned.
        {"name": "partitions-20m", "kind": "levels", "n": 20000000, "scale": 19, "days": 90, "thresholds": 29},
        # The repository's mid workload: 5e7 records over 2^20 vertices.
        {"name": "mid-50m", "kind": "edges", "graph": "rmat", "n": 50000000, "scale": 20, "days": 90, "M": 10,
         "hub": 0, "max_dt": -1, "kept": True},
        # A year with a hub in a large share of the records, the largest that a card holds three times over.
        {"name": "hub-200m", "kind": "edges", "graph": "rmat", "n": 200000000, "scale": 24, "days": 365, "M": 25,
         "hub": 1600000, "max_dt": -1, "kept": True},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rmat_scale(n, per_vertex):
    return max(1, min(24, int(math.ceil(math.log2(max(2.0, n / per_vertex))))))


def draw(rng):
    kind = rng.choice(["edges", "edges", "edges", "replay", "batch", "serve", "causal", "hyper", "levels"])
    M = rng.choice([2, 5, 10, 25, 50])
    if kind == "edges":
        graph = rng.choice(["rmat", "rmat", "bursts", "micros"])
        n = _log_uniform(rng, 500, 40_000_000 if graph == "rmat" else 4_000_000)
        case = {"kind": "edges", "graph": graph, "n": n, "days": rng.choice([1, 30, 90, 365]), "M": M,
                "hub": n // rng.choice([10, 100]) if graph == "rmat" and rng.random() < 0.3 else 0,
                "max_dt": rng.choice([-1, -1, -1, 3600, 86400]), "kept": rng.random() < 0.5}
        if graph == "rmat":
            case["scale"] = _rmat_scale(n, rng.uniform(4, 64))
        else:
            case["V"] = max(2, n // rng.randint(4, 64))
        return case
    if kind == "replay":
        n = _log_uniform(rng, 500, 1_000_000)
        return {"kind": "replay", "graph": "bursts", "n": n, "V": max(2, n // rng.randint(4, 64)), "days": 30, "M": M}
    if kind == "batch":
        return {"kind": "batch", "G": _log_uniform(rng, 2, 1000), "median": _log_uniform(rng, 1000, 20000),
                "sigma": round(rng.uniform(0.0, 1.5), 2), "lo": 500, "hi": 2000000, "M": M,
                "causal": rng.random() < 0.25}
    if kind == "serve":
        return {"kind": "serve", "requests": rng.randint(2, 64), "median": _log_uniform(rng, 1000, 70711),
                "sigma": round(rng.uniform(0.0, 1.42), 2), "lo": 1000, "hi": 2000000, "M": M}
    if kind == "causal":
        n = _log_uniform(rng, 500, 16_000_000)
        return {"kind": "causal", "n": n, "scale": _rmat_scale(n, rng.uniform(4, 64)), "days": rng.choice([30, 90]),
                "M": M, "thresholds": rng.choice([0, 8, 29])}
    if kind == "hyper":
        n = _log_uniform(rng, 500, 6_000_000)
        return {"kind": "hyper", "n": n, "V": max(2, n // rng.randint(4, 64)), "days": rng.choice([30, 90]), "M": M}
    n = _log_uniform(rng, 1000, 30_000_000)
    return {"kind": "levels", "n": n, "scale": _rmat_scale(n, rng.uniform(4, 64)), "days": 90,
            "thresholds": rng.choice([1, 8, 29])}


# ---------------------------------------------------------------- inputs
class _Gen:
    """Seeded draws on the GPU."""

    def __init__(self, seed, dev):
        self.g = torch.Generator(device=dev)
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
        self.dev = dev

    def unif(self, n):
        return torch.rand(n, generator=self.g, device=self.dev)

    def below(self, n, k):
        return torch.randint(0, int(k), (n,), generator=self.g, device=self.dev)

    def exp_int(self, n, mean):
        """Exponential gaps in whole seconds."""
        return torch.rand(n, generator=self.g, device=self.dev).neg_().log1p_().mul_(-float(mean)).floor_().long()

    def perm(self, V):
        return torch.randperm(int(V), generator=self.g, device=self.dev).to(torch.int32)


def _chung_lu(V, gamma=2.1):
    w = np.cumsum(np.arange(1, V + 1, dtype=np.float64) ** (-1.0 / (gamma - 1.0)))
    return w / w[-1]


def _pick(cdf, u, V):
    return torch.searchsorted(cdf, u.double()).clamp_(max=V - 1).to(torch.int32)


def _bursts(gen, n, V, days):
    """Conversations: bursts of 5..50 records around one person, gaps of a minute on average."""
    T = int(days) * DAY
    nb = n // 5 + 1
    size = 5 + gen.below(nb, 46)
    ends = torch.cumsum(size, 0)
    b = torch.searchsorted(ends, torch.arange(n, device=gen.dev), right=True)
    gap = gen.exp_int(n, 60.0)
    run = torch.cumsum(gap, 0)
    first = (ends - size)[b]
    t = gen.below(nb, T)[b] + run - run[first.clamp_(max=n - 1)]
    cdf = torch.from_numpy(_chung_lu(V)).to(gen.dev)
    u = _pick(cdf, gen.unif(nb), V)[b]
    x = _pick(cdf, gen.unif(n), V)
    x = torch.where(x == u, (x + 1) % V, x)
    perm = gen.perm(V)
    u, x = perm[u.long()], perm[x.long()]
    flip = gen.unif(n) < 0.5
    return torch.where(flip, x, u), torch.where(flip, u, x), t % T


def _rmat(gen, n, scale, days, hub=0):
    """R-MAT endpoints, relabelled; per pair a session of self-exciting gaps; `hub` endpoints moved to one vertex."""
    T, V = int(days) * DAY, 1 << int(scale)
    s = torch.zeros(n, dtype=torch.int32, device=gen.dev)
    d = torch.zeros(n, dtype=torch.int32, device=gen.dev)
    for _ in range(int(scale)):
        u = gen.unif(n)
        s.mul_(2).add_(u >= 0.76)
        d.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    d = torch.where(s == d, d ^ 1, d)
    if hub:
        i = gen.below(int(hub), n)
        side = gen.unif(int(hub)) < 0.5
        a, b = i[side], i[~side]
        s[a[d[a] != 0]] = 0
        d[b[s[b] != 0]] = 0
    key, order = torch.sort((s.long() << int(scale)) | d.long(), stable=True)
    start = torch.ones(n, dtype=torch.bool, device=gen.dev)
    start[1:] = key[1:] != key[:-1]
    del key
    group = torch.cumsum(start, 0) - 1
    first = torch.nonzero(start).view(-1)
    gap = torch.where(gen.unif(n) < 0.7, gen.exp_int(n, 30.0), gen.exp_int(n, 300.0))
    run = torch.cumsum(gap, 0)
    del gap
    tt = gen.below(first.numel(), T)[group] + run - run[first][group]
    del run, group, first, start
    t = torch.empty_like(tt)
    t[order] = tt % T
    del tt, order
    perm = gen.perm(V)
    return perm[s.long()], perm[d.long()], t


def _records(gen, case):
    n = int(case["n"])
    if case.get("graph", "rmat") == "rmat":
        s, d, t = _rmat(gen, n, case["scale"], case["days"], case.get("hub", 0))
        return s, d, t, 1 << int(case["scale"])
    s, d, t = _bursts(gen, n, int(case["V"]), case["days"])
    if case["graph"] == "micros":
        t = t * 1_000_000 + gen.below(n, 1_000_000)
    return s, d, t, int(case["V"])


def _sizes(count, median, sigma, lo, hi):
    """Lognormal sizes, one at each of `count` even quantiles, clipped."""
    q = (torch.arange(int(count), dtype=torch.float64) + 0.5) / int(count)
    z = (math.sqrt(2.0) * torch.erfinv(2 * q - 1)).numpy()
    return np.clip(np.rint(median * np.exp(sigma * z)), lo, hi).astype(np.int64)


def _shuffled_sizes(case, count, seed):
    sizes = _sizes(count, case["median"], case["sigma"], case["lo"], case["hi"])
    return np.random.default_rng(int(seed)).permutation(sizes)


def _zeroed(outputs):
    """Output buffers as a caller keeps them: their entries past a call's counts stay 0."""
    for x in outputs.t.values():
        x.zero_()
    return outputs


def _bytes(k, dev):
    return torch.empty(int(k), dtype=torch.uint8, device=dev)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = _Gen(seed, dev)
    kind, st = case["kind"], {"kind": case["kind"]}
    thr = PAPER_THRESHOLDS[-int(case["thresholds"]):] if case.get("thresholds") else None
    if kind in ("edges", "causal", "replay"):
        s, d, t, V = _records(gen, case)
        n, M = int(case["n"]), int(case["M"])
        st.update(ins=(s, d, t), M=M, V=V, n=n, thr=thr, max_dt=int(case.get("max_dt", -1)),
                  out=_zeroed(ce.Outputs(n, M, dev)), ws=None)
        if case.get("kept", True):
            st["ws"] = _bytes(ce.workspace_bytes(n, V, M, thresholds=thr), dev)
        if kind == "replay":
            st["hdr"] = torch.zeros(ce.hdr_words(1), dtype=torch.int64, device=dev)

            def enqueue():
                ce.cluster_edges_async(s, d, t, M, V, st["out"], st["ws"], st["hdr"], time_bits=32,
                                       stream=torch.cuda.current_stream())
            enqueue()
            graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream(device=dev)
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                with torch.cuda.graph(graph, stream=side):
                    enqueue()
            torch.cuda.synchronize()
            st["graph"] = graph
    elif kind == "batch":
        M, G = int(case["M"]), int(case["G"])
        sizes = _shuffled_sizes(case, G, seed)
        eoff = np.zeros(G + 1, dtype=np.int64)
        np.cumsum(sizes, out=eoff[1:])
        vs = np.maximum(2, sizes // 20)
        voff = np.zeros(G + 1, dtype=np.int64)
        np.cumsum(vs, out=voff[1:])
        n = int(eoff[-1])
        # bursts over one graph of the batch's mean density, folded into each graph's own vertices
        s, d, t = _bursts(gen, n, int(vs.max()), 30)
        g = torch.repeat_interleave(torch.arange(G, device=dev), torch.from_numpy(sizes).to(dev))
        v = torch.from_numpy(vs).to(dev)[g].to(torch.int32)
        s, d = s % v, d % v
        d = torch.where(s == d, (d + 1) % v, d)
        st.update(ins=(s, d, t), eoff=eoff, voff=voff, M=M, causal=bool(case["causal"]),
                  out=_zeroed(ce.batch_outputs(eoff, M, dev)), ws=_bytes(ce.batch_workspace_bytes(eoff, voff, M), dev))
    elif kind == "serve":
        M = int(case["M"])
        sizes = _shuffled_sizes(case, case["requests"], seed)
        caps = [ce.max_clusters(int(k), M) for k in sizes]
        out = _zeroed(ce.Outputs(int(sizes.sum()), M, dev, clusters=sum(caps), rows=int(sizes.sum())))
        reqs, r0, c0 = [], 0, 0
        for k, cap in zip(sizes, caps):
            k = int(k)
            scale = _rmat_scale(k, 16)
            host = [x.cpu().pin_memory() for x in _rmat(gen, k, scale, 90)]
            reqs.append(([x.numpy() for x in host], 1 << scale, out.region(r0, r0, c0, k, M), host))
            r0, c0 = r0 + k, c0 + cap
        torch.cuda.synchronize()
        # room for the whole burst twice over: admission is not what is waited for
        work = sum(ce.server_request_bytes(int(k), 1, M) for k in sizes)
        st.update(reqs=reqs, M=M, out=out, dev=dev, server=ce.Server(
            2 * work + (1 << 30), workers=3, max_inflight=max(64, len(reqs))))
    elif kind == "hyper":
        M, n, V = int(case["M"]), int(case["n"]), int(case["V"])
        s, d, t = _bursts(gen, n, V, case["days"])
        k = (2.0 * torch.exp(torch.randn(n, generator=gen.g, device=dev))).round_().clamp_(1, 64).long()
        off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
        torch.cumsum(k + 1, 0, out=off[1:])
        nnz = int(off[-1])
        cdf = torch.from_numpy(_chung_lu(V)).to(dev)
        mem = gen.perm(V)[_pick(cdf, gen.unif(nnz), V).long()]
        mem[off[:-1]] = s
        mem[off[:-1] + 1] = d
        st.update(ins=(mem, off, t), M=M, V=V, out=_zeroed(ce.Outputs(n, M, dev)),
                  ws=_bytes(ce.hyper_workspace_bytes(n, nnz, V, M), dev))
    else:
        s, d, t, V = _records(gen, case)
        n = int(case["n"])
        r = ce.cluster_edges(s, d, t, 10, V)
        st.update(ins=(r.msf_tail.clone(), r.msf_head.clone(), r.msf_w.clone()), n=n, thr=thr,
                  labels=torch.zeros(len(thr) * n, dtype=torch.int32, device=dev))
    return st


# ---------------------------------------------------------------- one pass
def _all(counts, st, discrete=False):
    """The counts, and the buffers that hold the outputs (whole, so that their shapes do not depend on the data)."""
    return [counts, {f: x for f, x in st["out"].t.items() if discrete or not f.startswith("dd_")}]


def run(st):
    kind = st["kind"]
    if kind == "edges":
        r = ce.cluster_edges(*st["ins"], st["M"], st["V"], outputs=st["out"], workspace=st["ws"], max_dt=st["max_dt"])
        return _all((r.m, r.n_clusters, r.n_labels), st)
    if kind == "causal":
        r = ce.cluster_edges(*st["ins"], st["M"], st["V"], outputs=st["out"], workspace=st["ws"], causal=True,
                             thresholds=st["thr"])
        return _all((r.m, r.n_clusters, r.n_labels), st, st["thr"] is not None)
    if kind == "replay":
        st["graph"].replay()
        return _all(st["hdr"], st)
    if kind == "batch":
        r = ce.cluster_batch(*st["ins"], st["eoff"], st["voff"], st["M"], outputs=st["out"], workspace=st["ws"],
                             causal=st["causal"])
        return _all((r.m, r.n_clusters, r.n_labels, r.row_offsets, r.cluster_offsets), st)
    if kind == "serve":
        srv, tickets, counts = st["server"], [], []
        for (s, d, t), V, out, _ in st["reqs"]:
            tickets.append(srv.submit(s, d, t, st["M"], V, outputs=out, device=st["dev"]))
        for k in tickets:
            r = srv.poll(k, wait=True)
            if r.status != ce.CE_OK:
                raise RuntimeError(r.error)
            counts.append((r.result.m, r.result.n_clusters, r.result.n_labels))
        return _all(np.array(counts, dtype=np.int64), st)
    if kind == "hyper":
        r = ce.cluster_hyperedges(*st["ins"], st["M"], st["V"], outputs=st["out"], workspace=st["ws"])
        return _all((r.m, r.n_clusters, r.n_labels), st)
    return ce.level_components(*st["ins"], st["n"], st["thr"], labels=st["labels"])


# ---------------------------------------------------------------- what a pass cannot do without
def _records_of(case):
    if case["kind"] in ("batch", "serve"):
        k = case["G"] if case["kind"] == "batch" else case["requests"]
        return int(_sizes(k, case["median"], case["sigma"], case["lo"], case["hi"]).sum())
    return int(case["n"])


def work(case):
    """Inputs once, outputs once; there is no floating point on the path."""
    n = _records_of(case)
    if case["kind"] == "levels":
        return {"bytes": 16.0 * n + 4.0 * n * int(case["thresholds"]), "flops": 0}
    given = 16.0 * n  # src, dst, t
    if case["kind"] == "hyper":
        given = 16.0 * n + 4.0 * 4.4 * n  # offsets, t, members
    rows, points = 36.0 * n, 16.0 * n  # forest and dendrogram rows; cluster, lambda and label of each record
    if case.get("thresholds"):
        rows += 8.0 * n
    return {"bytes": given + rows + points, "flops": 0}


def exact(case, seed):
    """Outputs are whole numbers throughout: they stay equal, and there is no rounding to hold against 64 bits."""
    return None
