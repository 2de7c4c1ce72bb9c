"""Products cut along k, where the last part has a single k (needs a GPU): the
oracle's bound in every kind of operands, and bits that differ from the uncut
division's, which shows that the cut ran (that these shapes are cut, and how, is
checked without a GPU by tests/host/launch_sim.cpp)."""

import numpy as np
import pytest

import oracle
import synth
from helpers import U32, U64, elementwise_bound, host_mats, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")


def device(x, dtype, pad):
    r, c = x.shape
    ld = -(-c // pad) * pad + (pad == 1 and c % 2 == 0)
    buf = torch.full((r, ld), float("nan"), dtype=dtype, device="cuda")
    buf[:, :c] = torch.from_numpy(np.ascontiguousarray(x)).to(dtype)
    return buf[:, :c]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("pad", [1, 16])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
def test_last_part_of_one_k(ta, tb, pad, dt):
    dtype = torch.float64 if dt == "f64" else torch.float32
    m, n = 33, 70
    for k in (12097, 16193, 19041):
        A, B, C = host_mats(synth.config_seed(1, 98) + k, m, n, k)
        if dt == "f32":
            A, B, C = (x.astype(np.float32).astype(np.float64) for x in (A, B, C))
        dA, dB = device(A.T if ta else A, dtype, pad), device(B.T if tb else B, dtype, pad)
        log(f"cut ta={ta} tb={tb} pad={pad} {dt} k={k}")
        outs = []
        for cfg in (None, 19):  # the cut product, and the uncut 32x32 division
            dC = device(C, dtype, pad)
            mg.gemm_ex(dA, dB, dC, 1.5, 0.5, transa=bool(ta), transb=bool(tb), cfg=cfg)
            torch.cuda.synchronize()
            outs.append(dC.double().cpu().numpy())
        assert not np.array_equal(outs[0], outs[1])
        ref = oracle.dgemm(1.5, A, B, 0.5, C)
        bound = elementwise_bound(1.5, A, B, 0.5, C, k, u=U32 if dt == "f32" else U64)
        for o in outs:
            assert (np.abs(o - ref) <= bound).all(), k
