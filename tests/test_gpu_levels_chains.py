"""Level components where joins make one long chain of links in any level, the last included: paths (also in random
order of ids), paths with a row that comes to the far end of the chain, caterpillars; expected labels by construction.
And the time of a row that walks a whole chain by itself against that of the chain."""
import time

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rows(shape, n):
    """Rows of one weight that join all n records."""
    i = torch.arange(n, device="cuda")
    if shape == "path":
        tl, hd = i[:-1], i[1:]
    elif shape == "backwards":
        tl, hd = i[:-1].flip(0), i[1:].flip(0)
    elif shape == "random ids":
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        q = torch.randperm(n, generator=g, device="cuda")
        tl, hd = q[:-1], q[1:]
    elif shape == "late":  # a path of the records from 1 on; then record 0 at its end
        tl, hd = torch.cat([i[1:-1], i[:1]]), torch.cat([i[2:], i[-1:]])
    elif shape == "bridges":  # 16 interleaved paths, each joined at its end to the start of the next
        k = min(16, n)
        c = i[:k - 1]
        tl, hd = torch.cat([i[:-k], c + 1]), torch.cat([i[k:], c + (n - 1 - c) // k * k])
    else:  # caterpillar: the smaller half are leaves of a path of the larger half
        h = n // 2
        tl, hd = torch.cat([i[h:-1], i[:h]]), torch.cat([i[h + 1:], h + i[:h]])
    return tl.int().contiguous(), hd.int().contiguous()


@pytest.mark.parametrize("n", [2, 3, 33, 34, 65, 700, 20_000, (1 << 21) - 1, (1 << 21) + 3])
@pytest.mark.parametrize("shape", ["path", "backwards", "random ids", "late", "bridges", "caterpillar"])
def test_one_component(shape, n):
    import paper_2311_10337_amd as ce
    tl, hd = rows(shape, n)
    assert len(tl) == n - 1
    w = torch.ones(n - 1, dtype=torch.int64, device="cuda")
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    for thr in ([1], [0, 1], [1, 5], [0, 1, 5], [0]):
        lab = ce.level_components(tl, hd, w, n, thr)
        for k, t in enumerate(thr):
            assert torch.equal(lab[k], ids if t < 1 else torch.zeros_like(ids)), (thr, k)


@pytest.mark.parametrize("thr", [[1, 2], [1, 2, 5]])
@pytest.mark.parametrize("n", [64, 20_001, (1 << 21) + 3])
def test_pairs_then_path(n, thr):
    import paper_2311_10337_amd as ce
    i = torch.arange(n - 1, device="cuda")
    order = torch.argsort(i % 2, stable=True)  # rows in ascending weight: the even ones first
    lab = ce.level_components(i[order].int(), (i + 1)[order].int(), (1 + i % 2)[order].contiguous(), n, thr)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    assert torch.equal(lab[0], ids // 2 * 2)
    assert not lab[1:].any()


@pytest.mark.parametrize("thr", [[1], [1, 5]])
def test_time_of_a_late_row(thr):
    import paper_2311_10337_amd as ce
    n = 1_000_000
    w = torch.ones(n - 1, dtype=torch.int64, device="cuda")
    ms = {}
    for shape in ("path", "late"):
        tl, hd = rows(shape, n)
        for rep in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            ce.level_components(tl, hd, w, n, thr)
            torch.cuda.synchronize()
            ms[shape] = (time.perf_counter() - t0) * 1e3
    print("[gpu-levels] %s %s" % (thr, ms), flush=True)
    assert ms["late"] < 100, ms
