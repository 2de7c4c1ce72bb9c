"""Exponents and slices of the split preparation at the edges of its loads
and of the number range (needs a GPU).

The default slice counts are cut from one fixed-point word, the others round
by round; both must give the oracle's integers exactly.  Shapes cover rows
that end inside a 4-long load, rows longer than a workgroup holds in
registers (k > 4096) and rows that are not 16-byte aligned (odd pitch).
"""

import numpy as np
import pytest

from helpers import to_dev
from oracle import split as osplit
from test_split_gpu import ALGOS, decode_workspace, mg, torch

pytestmark = pytest.mark.gpu


def wide(rng, rows, cols):
    """Values over the whole exponent range, subnormals and zeros included;
    some rows and columns all zero, one of subnormals only."""
    x = np.ldexp(rng.uniform(-1, 1, (rows, cols)), rng.integers(-60, 20, (rows, cols)))
    x *= np.ldexp(1.0, rng.integers(-400, 400, (rows, 1)))
    pick = rng.integers(0, 40, (rows, cols))
    x[pick == 0] = 0.0
    x[pick == 1] = np.ldexp(rng.uniform(-1, 1, (pick == 1).sum()), -1040)
    x[pick == 2] = np.ldexp(-1.0, rng.integers(-300, 300, (pick == 2).sum()))
    x[pick == 3] = np.nextafter(np.ldexp(1.0, rng.integers(-9, 9, (pick == 3).sum())), 0)
    x[rows // 2] = np.ldexp(rng.uniform(-1, 1, cols), -1050)
    x[:, cols // 3] = 0.0
    return x


@pytest.mark.parametrize("kind", ["i8", "bf16"])
@pytest.mark.parametrize("s", [None, 3, 8])
@pytest.mark.parametrize("shape,pad", [((3, 5, 2), 0), ((66, 63, 131), 3), ((5, 70, 4099), 1)])
def test_slices_over_the_number_range(kind, s, shape, pad):
    m, n, k = shape
    algo, bits = ALGOS[kind], osplit.SPLIT_BITS[kind]
    s = mg.split_default_slices(algo) if s is None else s
    rng = np.random.default_rng(1000 + m + n + k)
    A, B = wide(rng, m, k), wide(rng, k, n)
    dA = to_dev(np.pad(A, ((0, 0), (0, pad)), constant_values=9.0))[:, :k]
    dB = to_dev(np.pad(B, ((0, 0), (0, pad)), constant_values=9.0))[:, :n]
    L = mg.split_layout(algo, s, m, n, k)
    ws = torch.full((L["total_bytes"],), 0x5A, dtype=torch.uint8, device="cuda")
    mg.split_prepare(algo, s, dA, dB, ws)
    torch.cuda.synchronize()
    E, F, As, Bs = decode_workspace(ws, L, s, m, n, k)
    Eo, Fo = osplit.split_scales(A, 1), osplit.split_scales(B, 0)
    assert np.array_equal(E[:m], Eo) and (E[m:] == 0).all()
    assert np.array_equal(F[:n], Fo) and (F[n:] == 0).all()
    Ao, _ = osplit.split_slices(A, Eo, 1, s, bits)
    Bo, _ = osplit.split_slices(B, Fo, 0, s, bits)
    assert np.array_equal(As[:, :m, :k], Ao)
    assert np.array_equal(Bs[:, :n, :k], Bo.transpose(0, 2, 1))
    assert (As[:, m:, :] == 0).all() and (As[:, :, k:] == 0).all()
    assert (Bs[:, n:, :] == 0).all() and (Bs[:, :, k:] == 0).all()
