"""GPU parity of the base products that run in pieces along the contraction (batches of
few rows) and of the tile kernels that take over when the workspace has no room for the
pieces: rows, columns and contractions around the edges of the tiles (32 / 64 / 128 rows,
64 / 128 columns, 64-wide K-steps), ranks whose rows are and are not 16-byte aligned,
single and grouped calls, W as it is and transposed, with and without dropout.

Bar: 2e-2 against the fp64 reference (bf16 inputs, fp32 sums, one rounding), and a
repeated call is bit-identical.
"""
import numpy as np
import pytest

import oracle
from paper_2607_28848_amd import workloads as wl
from gpu_util import TOL_BF16, oracle_bwd, oracle_fwd, to_dev, to_host, train_mask_slices

pytestmark = pytest.mark.gpu


def _bits(t):
    import torch
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _segments(T, Tt, n_ad):
    """Decode rows, one prefill segment and a training segment split over two adapters."""
    segs, pos = [], 0
    n_dec = min(T - Tt, 5)
    for i in range(n_dec):
        segs.append((pos, 1, i % n_ad, 0))
        pos += 1
    if Tt:
        cut = max(1, Tt * 2 // 3)
        segs.append((pos, cut, 1 % n_ad, 1))
        pos += cut
        if Tt - cut:
            segs.append((pos, Tt - cut, 2 % n_ad, 1))
            pos += Tt - cut
    if T - pos:
        segs.append((pos, T - pos, 0, 0))
    return segs


CASES = [
    # T, T_t, K, N, r_max, ranks
    (1, 0, 1032, 72, 64, [16, 8, 64]),        # one decode row; K = 16 steps + 8, one ragged column tile
    (32, 0, 2056, 264, 16, [16, 8, 5]),       # a full 32-row tile
    (33, 20, 2048, 1000, 12, [12, 8, 5]),     # one row past it; rank rows of 24 bytes
    (65, 33, 4096, 1160, 64, [64, 33, 16]),   # one row past the 64-row tile, both rank steps
    (129, 64, 1544, 2056, 32, [32, 16, 7]),
    (260, 129, 2056, 1288, 16, [16, 8, 16]),  # several items and row tiles
]


@pytest.mark.parametrize("wt", [False, True])
@pytest.mark.parametrize("T,Tt,K,N,r_max,ranks", CASES)
def test_pieces_and_tiles_against_reference(T, Tt, K, N, r_max, ranks, wt):
    import torch
    from paper_2607_28848_amd import dsv
    w = wl.custom(_segments(T, Tt, len(ranks)), ranks, K=K, N=N, r_max=r_max, name="pieces")
    shapes = [(K, N), (K, 2 * N)]  # a group of two on the same batch
    w.projections = [wl.Projection("p%d" % i, *s) for i, s in enumerate(shapes)]
    ts = [w.tensors(i, pad=np.nan) for i in range(2)]
    dev = [{k: to_dev(t.store[k], "bf16") for k in ("X", "W", "A", "B", "dY")} for t in ts]
    plan = dsv.segments_build(w.segments, w.n_tokens, w.ranks, w.scales, w.r_max, device="cuda")
    drops = [(0.1, 5, 1), (0.1, 5, 2)] if wt and Tt else None
    keep = [oracle.dropout_multipliers(Tt, k, *drops[i]) if drops else None for i, (k, _) in enumerate(shapes)]
    refs = []
    for i in range(2):
        w.projections = [wl.Projection("p", *shapes[i])]
        Yr, _ = oracle_fwd(w, ts[i], drop=keep[i])
        refs.append((Yr, oracle_bwd(w, ts[i], drop=keep[i]) if Tt else None))

    def run(ids, short):
        """Grouped forward and backward of projections ids; short: workspaces 256 bytes too
        small for the pieces, so the tile kernels run."""
        sh = [shapes[i] for i in ids]
        need = [dsv.fwd_grouped_workspace_bytes(plan, dsv.BF16, sh)]
        need += [dsv.bwd_grouped_workspace_bytes(plan, dsv.BF16, sh)] if Tt else []
        ws = [torch.empty(n - (256 if short else 0), dtype=torch.uint8, device="cuda") for n in need]
        dr = [drops[i] for i in ids] if drops else None
        out = dsv.cobatch_fwd_grouped(plan, [(dev[i]["X"], dev[i]["W"], dev[i]["A"], dev[i]["B"]) for i in ids],
                                      workspace=ws[0], dropouts=dr)
        grads = dsv.lora_bwd_grouped(
            plan, [(dev[i]["X"], dev[i]["W"], dev[i]["A"], dev[i]["B"], out[n][1], dev[i]["dY"])
                   for n, i in enumerate(ids)], workspace=ws[1], dropouts=dr,
            wts=[dev[i]["W"].t().contiguous() for i in ids] if wt else None) if Tt else []
        torch.cuda.synchronize()
        return out, grads

    fc = dsv.gemm_config(plan, dsv.BF16, K, N, 0)
    print("T=%d T_t=%d K=%d N=%d wt=%s: fwd %s" % (T, Tt, K, N, wt, fc), flush=True)
    # pieces are what is tested: every tile summed from pieces
    assert fc["split_tiles"] == fc["row_tiles"] * fc["col_tiles"] > 0
    for ids in ([0], [0, 1]):
        for short in (False, True):
            out, grads = run(ids, short)
            out2, grads2 = run(ids, short)
            for n, i in enumerate(ids):
                errs = {"Y": oracle.rel_err(to_host(out[n][0]), refs[i][0])}
                assert torch.equal(_bits(out[n][0]), _bits(out2[n][0]))
                if Tt:
                    _, dAr, dBr, dXr = refs[i][1]
                    errs["dX"] = oracle.rel_err(to_host(grads[n][2]), dXr)
                    assert torch.equal(_bits(grads[n][2]), _bits(grads2[n][2]))
                    dA, dB = to_host(grads[n][0]), to_host(grads[n][1])
                    for a, r in train_mask_slices(w):
                        errs["dA%d" % a] = oracle.rel_err(dA[a, :r], dAr[a, :r])
                        errs["dB%d" % a] = oracle.rel_err(dB[a, :, :r], dBr[a, :, :r])
                print("  ids %s short %s " % (ids, short) + ", ".join("%s=%.1e" % kv for kv in errs.items()), flush=True)
                for k, v in errs.items():
                    assert v <= TOL_BF16, (ids, short, k, v)


@pytest.mark.parametrize("Tt", [3073, 3300])
def test_half_tiles_match_whole_tiles(Tt):
    """A last partial wave of 256 x 256 tiles run as 128-row halves: 13 row tiles (the last
    one ends in its first half, or in its second) by 16 column tiles per projection, so
    groups of 2, 3 and 4 leave 160, 112 and 64 tiles of a 256-CU wave: whole, halved and
    halved.  Every projection's Y, h and dX are the same bits in each group, and within the
    bar on rows at the halves' and tiles' edges."""
    import torch
    from paper_2607_28848_amd import dsv
    segs = [(0, 200, 0, 1), (200, Tt - 300, 1, 1), (Tt - 100, 100, 2, 1)]
    K, N = 1024, 4096
    w = wl.custom(segs, [16, 8, 5], K=K, N=N, r_max=16, name="half")
    w.projections = [wl.Projection("p", K, N)]
    t = w.tensors(0, pad=np.nan)
    d = {k: to_dev(t.store[k], "bf16") for k in ("X", "W", "A", "B", "dY")}
    plan = dsv.segments_build(w.segments, w.n_tokens, w.ranks, w.scales, w.r_max, device="cuda")
    outs = []
    for n in (2, 3, 4):
        out = dsv.cobatch_fwd_grouped(plan, [(d["X"], d["W"], d["A"], d["B"])] * n)
        grads = dsv.lora_bwd_grouped(plan, [(d["X"], d["W"], d["A"], d["B"], out[0][1], d["dY"])] * n)
        torch.cuda.synchronize()
        outs.append([o[0] for o in out] + [o[1] for o in out])
        outs.append([g[2] for g in grads])
    for group in (outs[0::2], outs[1::2]):
        flat = [x for o in group for x in o if x.shape == group[0][0].shape]
        assert all(torch.equal(_bits(x), _bits(flat[0])) for x in flat)
    rows = np.unique(np.concatenate([np.arange(0, Tt, 211), [127, 128, 255, 256, 3071, 3072, Tt - 101, Tt - 1]]))
    rows = rows.astype(np.int32)
    Yr, _ = oracle_fwd(w, t, rows)
    assert oracle.rel_err(to_host(outs[0][0])[rows], Yr) <= TOL_BF16
    dXr = oracle_bwd(w, t, dx_rows=rows)[3]
    assert oracle.rel_err(to_host(outs[1][0])[rows], dXr) <= TOL_BF16


@pytest.mark.parametrize("T,K,N", [(705, 4096, 4096), (400, 4096, 14336), (320, 1024, 1024)])
def test_zero_B_is_the_same_base_whatever_the_grouping(T, K, N):
    """B = 0: Y is the same bits for one segment (nothing gathered), for every row on its own
    (all gathered) and for a mix, in the ordinary and the allocation-free forward, at sizes
    near the line between pieces and tiles."""
    import torch
    from paper_2607_28848_amd import dsv
    gen = torch.Generator(device="cuda").manual_seed(3)
    X, W, A = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((T, K), (N, K), (3, 16, K)))
    B = torch.zeros((3, N, 16), dtype=torch.bfloat16, device="cuda")
    tables = [[(0, T, 0, 0)], [(t, 1, t % 3, 0) for t in range(T)], [(0, 1, 2, 0), (1, 150, 1, 1), (151, T - 151, 0, 0)]]
    outs = {"fwd": [], "noalloc": []}
    for segs in tables:
        plan = dsv.segments_build(segs, T, [16, 8, 16], [2.0] * 3, 16, device="cuda")
        print("T=%d K=%d N=%d gathered %d: %s" % (T, K, N, plan.counts()["gathered_rows"],
                                                  dsv.gemm_config(plan, dsv.BF16, K, N, 0)), flush=True)
        outs["fwd"].append(dsv.cobatch_fwd(plan, X, W, A, B)[0])
        outs["noalloc"].append(dsv.cobatch_fwd_noalloc(plan, X, W, A, B, torch.empty_like(outs["fwd"][0]))[0])
    torch.cuda.synchronize()
    for ys in outs.values():
        assert all(torch.equal(_bits(y), _bits(ys[0])) for y in ys[1:])
        assert oracle.rel_err(to_host(ys[0][::37]), to_host(X[::37]) @ to_host(W).T) <= TOL_BF16


# T = T_t of groups of two 2056 x 2056 projections, and the tile of their pieces (both passes).
WIDE_PIECES = {290: (128, 128), 490: (128, 256)}


@pytest.mark.parametrize("drop", [False, True])
@pytest.mark.parametrize("T", sorted(WIDE_PIECES))
def test_wide_pieces_one_weight_transposed(T, drop):
    """The pieces' 128 x 128 and 128 x 256 tiles, with ragged rows, columns and contraction
    (2056 = 8 * 256 + 8 = 32 * 64 + 8), in a group whose backward has the transposed weight of its second
    projection only: two launches of pieces, NN and NT, and one sum over both.  dX also with
    both weights as they are and both transposed, against the reference each time."""
    import torch
    from paper_2607_28848_amd import dsv
    K = N = 2056
    w = wl.custom([(0, 100, 0, 1), (100, 29, 1, 1), (129, T - 129, 2, 1)], [12, 8, 5], K=K, N=N, r_max=12, name="wide")
    w.projections = [wl.Projection("p%d" % i, K, N) for i in range(2)]
    ts = [w.tensors(i, pad=np.nan) for i in range(2)]
    d = [{k: to_dev(t.store[k], "bf16") for k in ("X", "W", "A", "B", "dY")} for t in ts]
    wt = [x["W"].t().contiguous() for x in d]
    plan = dsv.segments_build(w.segments, T, w.ranks, w.scales, w.r_max, device="cuda")
    drops = [(0.1, 5, 1), (0.1, 5, 2)] if drop else None
    keep = [oracle.dropout_multipliers(T, K, *drops[i]) if drop else None for i in range(2)]
    w.projections = w.projections[:1]
    print("T=%d drop=%s" % (T, drop), flush=True)
    out = dsv.cobatch_fwd_grouped(plan, [(x["X"], x["W"], x["A"], x["B"]) for x in d], dropouts=drops)
    grads = {}
    for wts in ((None, wt[1]), (None, None), (wt[0], wt[1])):
        grads[tuple(x is not None for x in wts)] = dsv.lora_bwd_grouped(
            plan, [(x["X"], x["W"], x["A"], x["B"], o[1], x["dY"]) for x, o in zip(d, out)], dropouts=drops, wts=list(wts))
    torch.cuda.synchronize()
    for i in range(2):
        errs = {"Y": oracle.rel_err(to_host(out[i][0]), oracle_fwd(w, ts[i], drop=keep[i])[0])}
        _, dAr, dBr, dXr = oracle_bwd(w, ts[i], drop=keep[i])
        for which, g in grads.items():
            errs["dX %s %s" % which] = oracle.rel_err(to_host(g[i][2]), dXr)
            dA, dB = to_host(g[i][0]), to_host(g[i][1])
            for a, r in train_mask_slices(w):
                errs["dA%d %s %s" % ((a,) + which)] = oracle.rel_err(dA[a, :r], dAr[a, :r])
                errs["dB%d %s %s" % ((a,) + which)] = oracle.rel_err(dB[a, :, :r], dBr[a, :, :r])
        print("  p%d " % i + ", ".join("%s=%.1e" % kv for kv in errs.items()), flush=True)
        for k, v in errs.items():
            assert v <= TOL_BF16, (i, k, v)


# T_t, K, N, projections of a masked backward whose dX has half tiles, and the tiles that
# stay whole and the tiles halved of one launch.
MASKED_HALVES = [
    (3073, 1024, 4096, 2, 0, 104),   # halves only; the last row tile ends in its first half
    (3300, 1024, 4096, 2, 0, 104),   # ... in its second
    (2049, 4104, 512, 2, 256, 50),   # behind whole tiles, the last column tile 8 wide
    (5000, 4104, 2048, 1, 256, 84),  # a single call
]


@pytest.mark.parametrize("wt", [False, True])
@pytest.mark.parametrize("Tt,K,N,n,whole,halves", MASKED_HALVES)
def test_masked_half_tiles(Tt, K, N, n, whole, halves, wt):
    """Half tiles that mask the low-rank term (dX under dropout), adapter runs that begin and
    end inside halves: against the reference at the halves' and tiles' edges, and the same
    bits as whole tiles (a group of three, whose last wave is too full for halves)."""
    import torch
    from paper_2607_28848_amd import dsv
    segs = [(0, 200, 0, 1), (200, Tt - 300, 1, 1), (Tt - 100, 99, 2, 1), (Tt - 1, 1, 0, 1)]
    w = wl.custom(segs, [16, 8, 40], K=K, N=N, r_max=64, name="masked_half")
    t = w.tensors(0, pad=np.nan)
    d = {k: to_dev(t.store[k], "bf16") for k in ("X", "W", "A", "B", "dY")}
    plan = dsv.segments_build(w.segments, w.n_tokens, w.ranks, w.scales, w.r_max, device="cuda")
    drop = (0.1, 5, 1)
    _, H = dsv.cobatch_fwd(plan, d["X"], d["W"], d["A"], d["B"], dropout=drop)
    Wt = d["W"].t().contiguous() if wt else None
    print("T_t=%d K=%d N=%d n=%d wt=%s" % (Tt, K, N, n, wt), flush=True)

    def grads(m):
        return dsv.lora_bwd_grouped(plan, [(d["X"], d["W"], d["A"], d["B"], H, d["dY"])] * m, dropouts=[drop] * m,
                                    wts=[Wt] * m if wt else None)

    got = grads(n) + (grads(3) if n > 1 else [])
    torch.cuda.synchronize()
    for g in got[1:]:
        assert torch.equal(_bits(g[2]), _bits(got[0][2]))
    rows = np.unique(np.concatenate([np.arange(0, Tt, 307), [127, 128, 199, 200, 255, 256, 383, 384, Tt - 101, Tt - 100,
                                                             (Tt - 1) // 256 * 256, Tt - 2, Tt - 1]])).astype(np.int32)
    dXr = oracle_bwd(w, t, dx_rows=rows, drop=oracle.dropout_multipliers(Tt, K, *drop))[3]
    err = oracle.rel_err(to_host(got[0][2])[rows], dXr)
    print("  dX %.2e" % err, flush=True)
    assert err <= TOL_BF16


def test_one_wave_of_dx_same_bits_either_weight():
    """dX of 1007 rows over 141 K-steps, 92 tiles in halves: W as it is and transposed give
    the same bits, within the bar on rows at the tiles' edges."""
    import torch
    from paper_2607_28848_amd import dsv
    Tt, K, N = 1007, 5880, 9016
    w = wl.custom([(0, 300, 0, 1), (300, Tt - 300, 1, 1)], [16, 8], K=K, N=N, r_max=16, name="one_wave")
    t = w.tensors(0, pad=np.nan)
    d = {k: to_dev(t.store[k], "bf16") for k in ("X", "W", "A", "B", "dY")}
    plan = dsv.segments_build(w.segments, w.n_tokens, w.ranks, w.scales, w.r_max, device="cuda")
    c = dsv.gemm_config(plan, dsv.BF16, K, N, 1)
    print("dX %s" % c, flush=True)
    out = [dsv.lora_bwd_grouped(plan, [(d["X"], d["W"], d["A"], d["B"], None, d["dY"])], wts=wts)[0][2]
           for wts in (None, [d["W"].t().contiguous()])]
    torch.cuda.synchronize()
    assert torch.equal(_bits(out[0]), _bits(out[1]))
    rows = np.array([0, 127, 128, 255, 256, 299, 300, 767, 768, 1006], dtype=np.int32)
    assert oracle.rel_err(to_host(out[0])[rows], oracle_bwd(w, t, dx_rows=rows)[3]) <= TOL_BF16
