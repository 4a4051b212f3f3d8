"""GPU parity of the fp32 mode around the edges of its tiles: 32 rows and columns, chunks
of 64 along the contraction, 64 training rows per step of a token sum (runs of one adapter
past 256 rows, several training adapters), ranks of one and of two column tiles, rank rows
that are and are not 16-byte aligned, dropout, h kept and recomputed.

Bar: 1e-5 against the fp64 reference (fp32 products and sums over at most 1032 terms of
random sign: about sqrt(1032) 2^-24 = 2e-6 of the largest result); repeats bit-identical.
"""
import numpy as np
import pytest

import oracle
from paper_2607_28848_amd import workloads as wl
from gpu_util import TOL_F32, Run, oracle_bwd, oracle_fwd, to_host, train_mask_slices

pytestmark = pytest.mark.gpu

CASES = [
    # segments, ranks, r_max, K, N, dropout
    ([(0, 1, 0, 1)], [1], 1, 8, 8, 0.0),
    ([(0, 32, 0, 0), (32, 33, 1, 1)], [8, 16], 16, 64, 32, 0.0),
    ([(0, 31, 0, 0), (31, 1, 1, 0), (32, 65, 1, 1), (97, 3, 2, 1)], [8, 33, 5], 33, 72, 40, 0.1),
    ([(0, 300, 1, 1), (300, 40, 0, 0), (340, 64, 2, 1), (404, 90, 1, 1)], [16, 64, 30], 64, 520, 136, 0.0),
    # steps of a token sum packed from many short runs, from part of a long one, and from more than 64
    ([(i, 1, i % 2, 1) for i in range(150)] + [(150, 70, 0, 1), (220, 3, 1, 1), (223, 300, 0, 1), (523, 5, 1, 1),
                                               (528, 61, 0, 1)], [33, 5], 33, 72, 40, 0.1),
    ([(3 * i, 3, i % 3, 1) for i in range(70)], [16, 8, 3], 16, 64, 32, 0.0),
    ([(0, 20, 3, 0), (20, 129, 0, 1), (149, 1, 1, 0)], [32, 7, 8, 10], 34, 1032, 264, 0.3),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_f32_tile_edges(case):
    import torch
    segs, ranks, r_max, K, N, p = CASES[case]
    w = wl.custom(segs, ranks, K=K, N=N, dtype="f32", r_max=r_max, name="f32_edges")
    run = Run(w)
    Tt = w.train_tokens
    d = (p, 11, 3) if p else None
    drop = oracle.dropout_multipliers(Tt, K, *d) if p else None
    args = (run.plan, run.X, run.W, run.A, run.B)
    out = []
    for keep in (True, False):
        Y, H = run.dsv.cobatch_fwd(*args, keep_h=keep, dropout=d)
        out.append((Y,) + tuple(run.dsv.lora_bwd(*args, H, run.dY, dropout=d)))
    torch.cuda.synchronize()
    Y, dA, dB, dX = out[0]
    errs = {"Y": oracle.rel_err(to_host(Y), oracle_fwd(w, run.t, drop=drop)[0])}
    _, dAr, dBr, dXr = oracle_bwd(w, run.t, drop=drop)
    errs["dX"] = oracle.rel_err(to_host(dX), dXr)
    for a, r in train_mask_slices(w):
        errs["dA%d" % a] = oracle.rel_err(to_host(dA)[a, :r], dAr[a, :r])
        errs["dB%d" % a] = oracle.rel_err(to_host(dB)[a, :, :r], dBr[a, :, :r])
    print(" case %d: " % case + ", ".join("%s=%.1e" % kv for kv in errs.items()), flush=True)
    for k, v in errs.items():
        assert v <= TOL_F32, (k, v)
    for a, b in zip(*out):  # h recomputed: the same bits
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
