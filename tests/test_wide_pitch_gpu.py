"""Row pitches just under the direct-load rings' limits (needs a GPU): B and A^T
with rows 128 MiB apart, A and B^T with rows 16 MiB apart, give the bits of the
same values in tightly packed rows, in every one-k-group ring."""

import pytest

import synth
from helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mg = pytest.importorskip("paper_1602_08477_amd")


def spread_rows(x, pitch_bytes):
    """The values of x in rows ``pitch_bytes`` apart (the gaps are not written)."""
    r, c = x.shape
    buf = torch.empty((r - 1) * (pitch_bytes // x.element_size()) + c, dtype=x.dtype,
                      device="cuda")
    v = buf.as_strided((r, c), (pitch_bytes // x.element_size(), 1))
    v.copy_(x)
    return v


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_pitches_at_the_ring_limit(ta, tb, dt):
    dtype = torch.float64 if dt == "f64" else torch.float32
    m, n, k = 133, 144, 77
    A, B, C = (torch.from_numpy(synth.matrix(97, i, *s)).to(dtype).cuda()
               for i, s in enumerate(((k, m) if ta else (m, k), (n, k) if tb else (k, n), (m, n))))
    pad = 16 * A.element_size()
    wide = (spread_rows(A, (1 << (27 if ta else 24)) - pad),
            spread_rows(B, (1 << (24 if tb else 27)) - pad))
    flat = tuple(torch.nn.functional.pad(x, (0, -x.shape[1] % 4))[:, :x.shape[1]]
                 for x in (A, B))
    for cfg in (14, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24):
        outs = []
        for a, b in (wide, flat):
            c = C.clone()
            mg.gemm_ex(a, b, c, 1.5, 0.5, transa=bool(ta), transb=bool(tb), cfg=cfg)
            torch.cuda.synchronize()
            outs.append(c)
        log(f"pitch ta={ta} tb={tb} {dt} cfg={cfg}")
        assert torch.equal(*outs), cfg
