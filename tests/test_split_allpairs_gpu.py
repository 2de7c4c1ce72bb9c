"""Work division 16 of the split path (all slice pairs from one stage) against
division 12, bit for bit, on both sides of its refill rule (needs a GPU).

Early refill: up to 2048 tiles of 64x64, or slices of a tile group that fit an
L2; late refill: larger products, and k of more than one exact INT32 segment.
"""

import pytest

from helpers import to_dev
from test_split_gpu import ALGOS, mg, spread, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["i8", "bf16"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 65, 64), (129, 200, 65), (2100, 1090, 300),
                                   (2944, 2950, 130), (2944, 2950, 700), (70, 130, 19200)])
@pytest.mark.parametrize("beta", [0.0, 0.5])
def test_all_pairs_equals_ring(kind, shape, beta):
    m, n, k = shape
    algo = ALGOS[kind]
    s = mg.split_default_slices(algo)
    A, B, C = (to_dev(x) for x in spread(70 + k, m, n, k))
    ws = mg.split_workspace(algo, s, m, n, k)
    got, want = C.clone(), C.clone()
    mg.gemm_split(A, B, got, 1.25, beta, algo=algo, workspace=ws, cfg=16)
    mg.gemm_split(A, B, want, 1.25, beta, algo=algo, workspace=ws, cfg=12)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
