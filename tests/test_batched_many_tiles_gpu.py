"""A batch whose work list passes 2^24 tiles, more than one dispatch of 256
lanes per tile can hold (needs a GPU): one row of C over 2^24 + 2 tiles of
32 x 32, replayed from its graph and launched directly, equal to the exact
small-integer result at every element."""

import pytest

from helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")


def test_more_tiles_than_one_dispatch():
    n = (1 << 29) + 33
    table = mg.TuneTable.from_list(mg.F32, [2] * mg.TUNE_BUCKETS)  # 32 x 32 tiles
    A = torch.full((1, 1), 3.0, dtype=torch.float32, device="cuda")
    B = torch.arange(n, dtype=torch.int32, device="cuda").remainder_(1021).float().view(1, n)
    C = torch.ones(1, n, dtype=torch.float32, device="cuda")
    plan = mg.Plan(mg.F32, [mg.problem(A, B, C, 1.0, 2.0)], table)
    assert plan.stats()["tiles"] == (1 << 24) + 2
    want = torch.ones_like(C)
    for graph in (True, False, True):
        log(f"{plan.stats()['tiles']} tiles, graph={graph}")
        plan.launch(graph=graph)
        want.mul_(2.0).add_(B, alpha=3.0)
        torch.cuda.synchronize()
        assert torch.equal(C, want)
    plan.close()
