"""The 32x32 direct-load ring around the k from which its unrolled loop runs
(needs a GPU): every layout gives the register-staged 32x32 tile's bits (the
same sums in the same order) and meets the oracle's bound, from k = 1 through
partial k-steps to just past the change of kernel."""

import numpy as np
import pytest

import oracle
import synth
from helpers import U32, U64, elementwise_bound, host_mats, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")


def device(x, dtype):
    r, c = x.shape
    buf = torch.full((r, -(-c // 16) * 16), float("nan"), dtype=dtype, device="cuda")
    buf[:, :c] = torch.from_numpy(np.ascontiguousarray(x)).to(dtype)
    return buf[:, :c]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_short_k_ring(ta, tb, dt):
    f64 = dt == "f64"
    dtype, bk = (torch.float64, 16) if f64 else (torch.float32, 32)
    m, n = 70, 45
    for k in (1, bk - 1, bk, bk + 1, 3 * bk, 4 * bk, 5 * bk + 3, 7 * bk, 8 * bk - 1, 8 * bk,
              8 * bk + 1, 9 * bk):
        A, B, C = host_mats(synth.config_seed(1, 95) + k, m, n, k)
        if not f64:
            A, B, C = (x.astype(np.float32).astype(np.float64) for x in (A, B, C))
        log(f"short k ta={ta} tb={tb} {dt} k={k}")
        dA, dB = device(A.T if ta else A, dtype), device(B.T if tb else B, dtype)
        outs = []
        for cfg in (19, 4):
            dC = device(C, dtype)
            mg.gemm_ex(dA, dB, dC, 1.5, 0.5, transa=bool(ta), transb=bool(tb), cfg=cfg)
            torch.cuda.synchronize()
            outs.append(dC.double().cpu().numpy())
        assert np.array_equal(outs[0], outs[1]), k
        ref = oracle.dgemm(1.5, A, B, 0.5, C)
        bound = elementwise_bound(1.5, A, B, 0.5, C, k, u=U64 if f64 else U32)
        assert (np.abs(outs[0] - ref) <= bound).all(), k
