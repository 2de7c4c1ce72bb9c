"""Further cases for the LDS-poison check (see lds_poison_cases.py), long enough
in k that every staged kernel runs its unrolled main loop as well as the
remainder: each native work division in FP64 and FP32 on 16-byte aligned and on
unaligned rows, the other layouts, k of one to nine k-steps on the 32x32 ring,
products cut along k, batches with k up to 700, and the split tile with its
stage refilled under the products and after them.

Child usage: python tests/lds_poison_loops.py OUT.npz
"""

from __future__ import annotations

import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)
sys.path.insert(0, os.path.dirname(HERE))


def run(out_path: str) -> int:
    import numpy as np
    import torch

    import paper_1602_08477_amd as mg
    import synth
    from helpers import NAIVE_CFG, make_batch

    res = {}

    def put(name, t):
        torch.cuda.synchronize()
        res[name] = t.detach().cpu().numpy()
        print(name, flush=True)

    def rows(x, dtype, odd):
        r, c = x.shape
        ld = -(-c // 16) * 16 + odd
        buf = torch.full((r, ld), float("nan"), dtype=dtype, device="cuda")
        buf[:, :c] = torch.from_numpy(np.ascontiguousarray(x)).to(dtype)
        return buf[:, :c]

    m, n, k = 150, 97, 603
    A = synth.matrix(21, synth.STREAM_A, m, k)
    B = synth.matrix(21, synth.STREAM_B, k, n)
    C = synth.matrix(21, synth.STREAM_C, m, n)
    for dt in (torch.float64, torch.float32):
        for odd in (0, 1):
            for ta, tb in ((0, 0), (1, 0), (0, 1), (1, 1)):
                a = rows(A.T if ta else A, dt, odd)
                b = rows(B.T if tb else B, dt, odd)
                for cfg in range(mg.num_tile_cfgs()):
                    if cfg == NAIVE_CFG or (ta or tb) and cfg not in (2, 4, 5, 13, 15, 18, 19, 20,
                                                                      21, 22, 23, 26, 27, 29):
                        continue
                    c = rows(C, dt, odd)
                    mg.gemm_ex(a, b, c, 1.5, 0.5, transa=bool(ta), transb=bool(tb), cfg=cfg)
                    put(f"{dt}_{odd}_{ta}{tb}_{cfg}", c)
        for kk in (16, 50, 100, 130, 250, 260):
            c = rows(C, dt, 0)
            mg.gemm_ex(rows(A[:, :kk], dt, 0), rows(B[:kk], dt, 0), c, 1.0, 1.0, cfg=19)
            put(f"{dt}_k{kk}", c)
        lA = synth.matrix(22, synth.STREAM_A, 70, 12097)
        lB = synth.matrix(22, synth.STREAM_B, 12097, 45)
        for odd in (0, 1):  # cut along k
            c = torch.zeros(70, 45, dtype=dt, device="cuda")
            mg.gemm(rows(lA, dt, odd), rows(lB, dt, odd), c, 1.0, 0.0)
            put(f"{dt}_cut_{odd}", c)
        shapes = [tuple(int(x) for x in s) for s in synth.batch_shapes(23, 40, 1, 700)]
        views, flats, probs = make_batch(23, shapes, dtype=dt)
        mg.gemm_batched(probs, dtype=mg.F64 if dt == torch.float64 else mg.F32)
        put(f"{dt}_grouped", flats["C"])
        del views, flats, probs

    for algo in (mg.SPLIT_I8, mg.SPLIT_BF16):
        # early refill of one k segment; then more than 768 tiles and k > 2048: late
        for sm, sn, sk in ((200, 150, 2600), (1800, 1800, 2100)):
            g = torch.Generator(device="cuda").manual_seed(24)
            sA = torch.rand(sm, sk, dtype=torch.float64, device="cuda", generator=g) - 0.5
            sB = torch.rand(sk, sn, dtype=torch.float64, device="cuda", generator=g) - 0.5
            c = torch.zeros(sm, sn, dtype=torch.float64, device="cuda")
            mg.gemm(sA, sB, c, 1.0, 0.0, algo=algo)
            put(f"split_{algo}_{sm}", c)
    res["build_flags"] = np.array([mg.build_flags()], dtype=np.int32)
    np.savez(out_path, **res)
    return len(res)


if __name__ == "__main__":
    print(f"lds poison loops: {run(sys.argv[1])} outputs written", flush=True)
