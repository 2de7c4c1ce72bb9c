"""Products with few outputs and a long k, whose k range is cut over
workgroups: against the oracle's bound at the edges of the cut (a last part
of one k, parts of unequal length, outputs of one tile and of ragged tiles),
for both kinds of operands; the same bits on every run; C <- beta C semantics
through the adding kernel; and under stream capture, where the product runs
uncut."""

import numpy as np
import pytest

import oracle
import synth
from helpers import U32, U64, elementwise_bound, host_mats, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")

DT = {"f64": torch.float64, "f32": torch.float32}


def device(x, dtype, pad):
    r, c = x.shape
    ld = -(-c // pad) * pad + (pad == 1 and c % 2 == 0)
    buf = torch.full((r, ld), float("nan"), dtype=dtype, device="cuda")
    buf[:, :c] = torch.from_numpy(np.ascontiguousarray(x)).to(dtype)
    return buf[:, :c]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("pad", [1, 16])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_long_k_matches_oracle(ta, tb, pad, dt):
    dtype = DT[dt]
    for i, (m, n, k) in enumerate([(64, 64, 16384), (1, 3, 20001), (65, 33, 9985), (130, 70, 8193),
                                   (200, 200, 12288)]):
        A, B, C = host_mats(synth.config_seed(1, 80) + i, m, n, k)
        if dt == "f32":
            A, B, C = (x.astype(np.float32).astype(np.float64) for x in (A, B, C))
        log(f"long k ta={ta} tb={tb} pad={pad} {dt} {(m, n, k)}")
        dA, dB = device(A.T if ta else A, dtype, pad), device(B.T if tb else B, dtype, pad)
        ref = {b: oracle.dgemm(1.5, A, B, b, C) for b in (0.5, 0.0)}
        for beta in (0.5, 0.0):
            outs = []
            for _ in range(2):
                dC = device(C, dtype, pad)
                if beta == 0.0:
                    dC.fill_(float("nan"))  # not read
                mg.gemm_ex(dA, dB, dC, 1.5, beta, transa=bool(ta), transb=bool(tb))
                torch.cuda.synchronize()
                outs.append(dC.double().cpu().numpy())
            assert np.array_equal(outs[0], outs[1])
            bound = elementwise_bound(1.5, A, B, beta, C, k, u=U32 if dt == "f32" else U64)
            assert (np.abs(outs[0] - ref[beta]) <= bound).all(), (m, n, k, beta)


def test_long_k_under_capture_and_on_streams():
    """Captured, the product runs uncut (no allocation in the graph): every
    replay gives the uncut division's bits.  Two streams in turn give the same
    bits as one."""
    m, n, k = 96, 80, 16384
    A, B, C = host_mats(synth.config_seed(1, 85), m, n, k)
    dA, dB, C0 = (torch.from_numpy(x).cuda() for x in (A, B, C))
    uncut = C0.clone()
    mg.gemm(dA, dB, uncut, 1.0, 1.0, cfg=mg.pick_tile_cfg(m, n, k))
    eager = C0.clone()
    mg.gemm(dA, dB, eager, 1.0, 1.0)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    outs = [C0.clone() for _ in range(8)]
    torch.cuda.synchronize()
    for i, c in enumerate(outs):
        mg.gemm(dA, dB, c, 1.0, 1.0, stream=streams[i % 2])
    torch.cuda.synchronize()
    assert all(torch.equal(c, eager) for c in outs)
    dC = C0.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mg.gemm(dA, dB, dC, 1.0, 1.0)
    for _ in range(3):
        dC.copy_(C0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dC, uncut)
    assert torch.allclose(uncut, eager, rtol=1e-12, atol=1e-10)
