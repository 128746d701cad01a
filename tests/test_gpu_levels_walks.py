"""Level components on forests whose joins make long walks (paths, one level or several) and hot roots (stars), at sizes
below and above the change of records per thread; expected labels by construction."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 65, 20_000, (1 << 21) - 1, (1 << 21) + 3])
@pytest.mark.parametrize("shape", ["path", "star", "pairs then path"])
def test_walks(shape, n):
    import torch
    import paper_2311_10337_amd as ce
    i = torch.arange(n - 1, dtype=torch.int32, device="cuda")
    tl, hd = (torch.zeros_like(i) if shape == "star" else i), i + 1
    w = torch.ones(n - 1, dtype=torch.int64, device="cuda")
    if shape == "pairs then path":  # rows in ascending weight: the even ones first
        order = torch.argsort((i % 2).to(torch.int64), stable=True)
        tl, hd, w = tl[order].contiguous(), hd[order].contiguous(), (1 + i % 2).to(torch.int64)[order].contiguous()
    lab = ce.level_components(tl, hd, w, n, [0, 1, 2])
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    assert torch.equal(lab[0], ids)
    assert torch.equal(lab[1], ids // 2 * 2 if shape == "pairs then path" else torch.zeros_like(ids))
    assert not lab[2].any()
