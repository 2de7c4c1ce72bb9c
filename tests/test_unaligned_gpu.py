"""Operands at any element address: the register-staged tiles load 16-byte
chunks from rows of every pitch and base, read a row's last full chunk where
one would run past its end, and read rows shorter than a chunk element by
element.  Shapes at the edges of that rule (rows of 1 element up to one past a
tile), operands inside NaN-filled buffers (a read outside the matrix that
reaches a sum shows), C inside a canary buffer."""

import numpy as np
import pytest

import oracle
import synth
from helpers import U32, U64, elementwise_bound, host_mats, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")

SHAPES = [(1, 1, 1), (2, 3, 1), (3, 2, 2), (33, 1, 3), (5, 4, 4), (65, 5, 6), (31, 66, 33),
          (129, 127, 17), (64, 65, 31)]


def embed(x, dtype, shift, fill):
    """x as a view of odd pitch inside a ``fill``-filled buffer, ``shift``
    elements past its 16-byte aligned base; returns (view, buffer)."""
    r, c = x.shape
    ld = (c + 2) | 1
    buf = torch.full((shift + r * ld + 8,), fill, dtype=dtype, device="cuda")
    v = buf[shift:shift + r * ld].view(r, ld)[:, :c]
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)).to(dtype))
    return v, buf


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("cfg", [-1, 0, 4, 5, 7, 8, 10])
def test_unaligned_edges(cfg, ta, tb, dt):
    dtype = torch.float64 if dt == "f64" else torch.float32
    for i, (m, n, k) in enumerate(SHAPES):
        A, B, C = host_mats(synth.config_seed(1, 70) + i, m, n, k)
        if dt == "f32":
            A, B, C = (x.astype(np.float32).astype(np.float64) for x in (A, B, C))
        log(f"unaligned cfg={cfg} ta={ta} tb={tb} {dt} {(m, n, k)}")
        dA, _ = embed(A.T if ta else A, dtype, 1, float("nan"))
        dB, _ = embed(B.T if tb else B, dtype, 3, float("nan"))
        dC, buf = embed(C, dtype, 1, 12345.0)
        before = buf.clone()
        mg.gemm_ex(dA, dB, dC, 1.5, 0.5, transa=bool(ta), transb=bool(tb),
                   cfg=None if cfg < 0 else cfg)
        torch.cuda.synchronize()
        got = dC.double().cpu().numpy()
        ref = oracle.dgemm(1.5, A, B, 0.5, C)
        bound = elementwise_bound(1.5, A, B, 0.5, C, k, u=U32 if dt == "f32" else U64)
        assert (np.abs(got - ref) <= bound).all(), (m, n, k)
        outside = torch.ones_like(buf, dtype=torch.bool)
        outside[1:1 + m * ((n + 2) | 1)].view(m, -1)[:, :n] = False
        assert torch.equal(buf[outside], before[outside]), (m, n, k)


@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
def test_pitch_beyond_ring_offsets(ta, tb):
    """16-byte aligned rows 16 MiB apart: past what the direct-load rings
    address from a tile's corner, so a register-staged tile runs."""
    m, n, k = 5, 6, 4
    A, B, C = host_mats(synth.config_seed(1, 71), m, n, k)
    ld = (1 << 21) + 2

    def far(x):
        t = torch.full((x.shape[0], ld), float("nan"), dtype=torch.float64, device="cuda")
        t[:, :x.shape[1]] = torch.from_numpy(np.ascontiguousarray(x))
        return t[:, :x.shape[1]]

    dA, dB = far(A.T if ta else A), far(B.T if tb else B)
    ref = oracle.dgemm(1.5, A, B, 0.5, C)
    bound = elementwise_bound(1.5, A, B, 0.5, C, k)
    for cfg in (None, 19, 21, 23, 26):
        log(f"far pitch cfg={cfg} ta={ta} tb={tb}")
        dC = torch.from_numpy(C).cuda()
        mg.gemm_ex(dA, dB, dC, 1.5, 0.5, transa=bool(ta), transb=bool(tb), cfg=cfg)
        torch.cuda.synchronize()
        assert (np.abs(dC.cpu().numpy() - ref) <= bound).all(), cfg


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("pad", [1, 16])
def test_picked_division_gives_the_same_bits(pad, dt):
    """Shapes around the points where the work-division rule changes its
    mind, for operands of both kinds: the picked division's result is the
    32x32 register-staged tile's, bit for bit (one k group)."""
    dtype = torch.float64 if dt == "f64" else torch.float32
    for i, (m, n, k) in enumerate([(31, 33, 65), (511, 513, 96), (1023, 1009, 50), (777, 2053, 40),
                                   (1531, 1033, 47), (2600, 700, 33), (3001, 2999, 35),
                                   (4095, 4097, 17)]):
        if pad > 1 and mg.pick_tile_cfg(m, n, k, mg.F64 if dt == "f64" else mg.F32) >= 26:
            continue
        log(f"pick {dt} pad={pad} {(m, n, k)}")
        g = torch.Generator(device="cuda").manual_seed(100 + i)

        def mat(r, c):
            t = torch.empty(r, -(-c // pad) * pad + (pad == 1 and c % 2 == 0), dtype=dtype,
                            device="cuda").uniform_(-1, 1, generator=g)
            return t[:, :c]

        A, B, C = mat(m, k), mat(k, n), mat(m, n)
        one, two = C.clone(), C.clone()
        mg.gemm(A, B, one, 1.5, 0.5)
        mg.gemm(A, B, two, 1.5, 0.5, cfg=4)
        torch.cuda.synchronize()
        assert torch.equal(one, two), (m, n, k)
