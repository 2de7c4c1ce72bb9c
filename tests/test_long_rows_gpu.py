"""One row of 2^29 + 7 outputs (needs a GPU): more workgroups than a dispatch
holds in the smallest tiles, or in 128x128 tiles on 16 wavefronts.  The default
division and the 128x128 ones give the exact small-integer result, on rows that
the direct-load rings take and on rows that they don't."""

import pytest

from helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")


@pytest.mark.parametrize("pitch_step", [16, 1])
def test_rows_past_one_dispatch(pitch_step):
    n, k = (1 << 29) + 7, 2
    ld = -(-n // pitch_step) * pitch_step
    B = torch.empty(k, ld, dtype=torch.float32, device="cuda")[:, :n]
    j = torch.arange(n, dtype=torch.int32, device="cuda")
    B[0] = j.remainder(509)
    B[1] = j.remainder_(251)
    del j
    A = torch.zeros(1, 16, dtype=torch.float32, device="cuda")[:, :k]
    A[0, 0], A[0, 1] = 2.0, 3.0
    want = 2.0 * B[0] + 3.0 * B[1] + 4.0
    for cfg in (None, 13, 17, 21, 22):
        C = torch.ones(1, n, dtype=torch.float32, device="cuda")
        log(f"long row, pitch step {pitch_step}, cfg {cfg}")
        mg.gemm(A, B, C, 1.0, 4.0, cfg=cfg)
        torch.cuda.synchronize()
        assert torch.equal(C[0], want), cfg


def test_rows_past_one_dispatch_f64():
    """The FP64 128x128 ring, whose 16 wavefronts do not fit the dispatch."""
    n = (1 << 29) + 7
    B = torch.arange(n, dtype=torch.int32, device="cuda").remainder_(1021).double().view(1, n)
    buf = torch.empty(1, n + 1, dtype=torch.float64, device="cuda")  # even pitch
    buf[:, :n] = B
    del B
    B, A = buf[:, :n], torch.full((1, 2), 3.0, dtype=torch.float64, device="cuda")[:, :1]
    for cfg in (None, 21):
        C = torch.ones(1, n, dtype=torch.float64, device="cuda")
        log(f"long row f64, cfg {cfg}")
        mg.gemm(A, B, C, 1.0, 2.0, cfg=cfg)
        torch.cuda.synchronize()
        assert bool((C - 3.0 * B == 2.0).all()), cfg
