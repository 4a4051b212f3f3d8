"""Which kernels a call launches, on the CPU: the library's host code is built with the
launchers and the HIP calls replaced by stubs that write down each launch
(launch_recorder.cpp) for a device of 256 compute units, and called through the binding
with addresses that nothing reads."""
import ctypes
import importlib.util
import os
import re
import subprocess

import pytest

from paper_2607_28848_amd import build as pkg_build

HERE = os.path.dirname(os.path.abspath(__file__))
BUF = 1 << 30   # an operand's address
WS = 1 << 40    # the workspace's
SCRATCH = 64 << 20


class Recorded:
    """The binding on the recording library: call(fn) -> (status, launches)."""

    def __init__(self, path):
        old = os.environ.get("DSV_LIBRARY")
        os.environ["DSV_LIBRARY"] = path
        try:
            spec = importlib.util.spec_from_file_location("dsv_recorded", os.path.join(pkg_build.PKG, "dsv.py"))
            self.dsv = importlib.util.module_from_spec(spec)
            spec.loader.exec_module(self.dsv)
        finally:
            if old is None:
                del os.environ["DSV_LIBRARY"]
            else:
                os.environ["DSV_LIBRARY"] = old
        self.lib = self.dsv.lib_handle()
        self.lib.recorder_log.restype = ctypes.c_char_p
        self.lib.recorder_scratch.restype = ctypes.c_void_p

    def plan(self, segs, ranks, r_max):
        p = self.dsv.segments_build(segs, sum(s[1] for s in segs), ranks, [2.0] * len(ranks), r_max)
        assert self.lib.dsv_plan_upload(p.handle, WS, p.meta_bytes, None) == self.dsv.OK
        return p

    def call(self, fn, *args):
        self.lib.recorder_clear()
        rc = fn(*args)
        out = []
        for l in self.lib.recorder_log().decode().splitlines():
            kind, *kv = l.split()
            out.append(dict({"kind": kind}, **{k: int(v) for k, v in (x.split("=") for x in kv)}))
        return rc, out

    def fwd(self, p, K, N, dtype=0, short=0):
        n = self.dsv.fwd_workspace_bytes(p, dtype, K, N) - short
        return self.call(self.lib.dsv_cobatch_fwd, p.handle, dtype, K, N, BUF, BUF, BUF, BUF, BUF, BUF, WS, n, None)

    def noalloc(self, p, K, N):
        return self.call(self.lib.dsv_cobatch_fwd_noalloc, p.handle, 0, K, N, BUF, BUF, BUF, BUF, BUF, BUF, None)

    def fwd_grouped(self, p, shapes, dropout=False):
        n = self.dsv.fwd_grouped_workspace_bytes(p, 0, shapes)
        pr = b"".join(self.dsv._FWD_PACK(K, N, BUF, BUF, BUF, BUF, BUF, BUF, 0, 0, 0) for K, N in shapes)
        if dropout:
            drops = (self.dsv.Dropout * len(shapes))(*[self.dsv.Dropout(0.05, 1, i, None) for i in range(len(shapes))])
            return self.call(self.lib.dsv_cobatch_fwd_grouped_dropout, p.handle, 0, len(shapes), pr, drops, WS, n, None)
        return self.call(self.lib.dsv_cobatch_fwd_grouped, p.handle, 0, len(shapes), pr, WS, n, None)

    def bwd_grouped(self, p, shapes, wt=True, dropout=False, short=0):
        n = self.dsv.bwd_grouped_workspace_bytes(p, 0, shapes) - short
        pr = b"".join(self.dsv._BWD_PACK(K, N, BUF, BUF, BUF, BUF, BUF, BUF, BUF, BUF, BUF, BUF if wt else 0,
                                         0, 0, 0, 0, 0) for K, N in shapes)
        args = (p.handle, 0, len(shapes), pr, 0)
        if not dropout:
            return self.call(self.lib.dsv_lora_bwd_grouped, *args, WS, n, None)
        drops = (self.dsv.Dropout * len(shapes))(*[self.dsv.Dropout(0.05, 1, i, None) for i in range(len(shapes))])
        return self.call(self.lib.dsv_lora_bwd_grouped_dropout, *args, drops, WS, n, None)


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rec") / "librecorded.so")
    srcs = [os.path.join(pkg_build.CSRC, s) for s in pkg_build.HOST_SOURCES] + [os.path.join(HERE, "launch_recorder.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(pkg_build.ROCM, "include"), "-I", os.path.join(pkg_build.ROOT, "include"),
                    "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", so] + srcs, check=True)
    return Recorded(so)


def _base(launches):
    """How the base product is summed: its launches without addresses and without the shrink."""
    return [tuple((k, v) for k, v in l.items() if k not in ("shrink", "part", "h_part", "h_bytes"))
            for l in launches if re.match("part|gemm|group", l["kind"])]


@pytest.mark.parametrize("K,N", [(4096, 4096), (4096, 14336), (14336, 4096), (1024, 1024), (520, 776)])
def test_base_product_does_not_depend_on_the_grouping(rec, K, N):
    """Tables of as many rows, one segment or every row on its own (all gathered), sum the
    base product alike in every forward, masked training rows or none: with B = 0 their
    results are then the same bits."""
    refused = 0
    for T in list(range(1, 258, 37)) + list(range(260, 1400, 29)):
        a = rec.plan([(0, T, 0, 0)], [16, 16], 16)
        b = rec.plan([(t, 1, t % 2, 0) for t in range(T)], [16, 16], 16)
        assert b.counts()["gathered_rows"] == T
        for what, call in (("single", lambda p: rec.fwd(p, K, N)), ("noalloc", lambda p: rec.noalloc(p, K, N)),
                           ("group", lambda p: rec.fwd_grouped(p, [(K, N), (K, 8 * (N // 16))]))):
            (ra, la), (rb, lb) = call(a), call(b)
            if what == "noalloc" and rec.dsv.ERR_SIZE in (ra, rb):
                refused += 1  # the gathered rows' terms alone exceed the scratch
                continue
            assert ra == rb == rec.dsv.OK
            assert _base(la) and _base(la) == _base(lb), (what, T, la, lb)
        c = rec.plan([(0, T - T // 2, 0, 0), (T - T // 2, T // 2, 1, 1)], [16, 16], 16)
        for shapes in ([(K, N)], [(K, N), (K, 8 * (N // 16))]):
            assert _base(rec.fwd_grouped(c, shapes, dropout=True)[1]) == _base(rec.fwd_grouped(a, shapes)[1])
    assert refused < 40


def test_noalloc_pieces_stay_inside_the_scratch(rec):
    """Pieces of the allocation-free forward lie within the 64 MiB scratch, however the
    rows are grouped, up to the largest that fit."""
    base, most = rec.lib.recorder_scratch(), 0
    for K, N in ((4096, 4096), (4096, 14336), (14336, 4096), (28672, 8192), (65536, 8192)):
        for T in (1, 33, 200, 256, 365, 600, 620, 638, 655, 768):
            for p in (rec.plan([(0, T, 0, 0)], [64], 64), rec.plan([(t, 1, t % 2, 0) for t in range(T)], [64] * 2, 64)):
                rc, launches = rec.noalloc(p, K, N)
                for l in launches:
                    if l["kind"] == "part":
                        ends = [l["part"] + l["bytes"] - base, l["h_part"] + l["h_bytes"] - base]
                        assert l["part"] >= base and l["h_part"] >= base and max(ends) <= SCRATCH, (K, N, T, l)
                        most = max(most, *ends)
    assert most > SCRATCH * 7 // 8


# Calls timed both ways on MI355X (one segment): projections, rows, microseconds in pieces
# and in tiles.
TIMED = [
    # forward, one projection
    ("fwd", [(64, 131072)], 256, 73.6, 25.2), ("fwd", [(1024, 32768)], 128, 34.2, 23.0),
    ("fwd", [(512, 14336)], 256, 23.6, 14.4),
    ("fwd", [(4096, 131072)], 128, 311.8, 202.4), ("fwd", [(4096, 14336)], 304, 69.0, 58.3),
    ("fwd", [(5120, 14336)], 380, 109.7, 87.4), ("fwd", [(8192, 28672)], 76, 125.2, 209.9),
    ("fwd", [(28672, 8192)], 240, 150.1, 179.1), ("fwd", [(4096, 4096)], 360, 30.3, 45.5),
    ("fwd", [(8192, 512)], 8192, 114.2, 101.5), ("fwd", [(14336, 512)], 6144, 140.4, 120.8),
    ("fwd", [(4096, 512)], 16384, 113.8, 98.5), ("fwd", [(4096, 256)], 32768, 160.3, 134.7),
    ("fwd", [(4096, 256)], 2500, 29.0, 43.5),
    # ... two and three
    ("fwd", [(4096, 64)] * 3, 16384, 217.7, 178.0), ("fwd", [(8192, 28672)] * 2, 209, 315.5, 248.6), ("fwd", [(4096, 14336)] * 2, 90, 61.9, 100.2),
    ("fwd", [(4096, 14336)] * 2, 142, 82.5, 113.5), ("fwd", [(4096, 14336)] * 2, 235, 80.7, 104.8), ("fwd", [(5120, 28672)] * 2, 256, 215.6, 144.0),
    ("fwd", [(4096, 14336)] * 2, 515, 198.5, 155.2), ("fwd", [(4096, 4096)] * 2, 60, 22.8, 60.2),
    # backward
    ("bwd", [(64, 2048)], 16384, 54.0, 73.1), ("bwd", [(4368, 848)] * 3, 221, 42.8, 55.4),
    ("bwd", [(1024, 3072)] * 2, 3399, 99.6, 84.0), ("bwd", [(5120, 64), (648, 28672)], 3, 39.4, 531.8),
    ("bwd", [(14336, 512)], 250, 42.7, 33.9), ("bwd", [(14336, 4096)], 323, 91.2, 71.8),
    ("bwd", [(28672, 1024)], 248, 57.4, 46.1), ("bwd", [(4096, 14336)], 240, 63.8, 72.2),
    ("bwd", [(4096, 14336)] * 2, 436, 142.1, 192.4), ("bwd", [(28672, 5120)] * 2, 240, 282.1, 207.1),
]


@pytest.mark.parametrize("what,shapes,T,pieces_us,tiles_us", TIMED)
def test_the_faster_of_pieces_and_tiles_runs(rec, what, shapes, T, pieces_us, tiles_us):
    p = rec.plan([(0, T, 0, int(what == "bwd"))], [16], 16)
    rc, launches = rec.fwd_grouped(p, shapes) if what == "fwd" else rec.bwd_grouped(p, shapes)
    kinds = {l["kind"] for l in launches if re.match("part|gemm|group", l["kind"])}
    assert rc == rec.dsv.OK and (kinds == {"part"}) == (pieces_us < tiles_us), (kinds, launches)


@pytest.mark.parametrize("T,K,N", [(1007, 9016, 5880), (3908, 8760, 1776), (8128, 8552, 1008)])
def test_one_wave_over_a_long_contraction_is_split(rec, T, K, N):
    """Forwards timed in 131, 140 and 155 us with their one partial wave split in two, in 161, 169
    and 172 with halves."""
    (rc, launches) = rec.fwd(rec.plan([(0, T, 0, 0)], [16], 16), K, N)
    l, = [l for l in launches if re.match("part|gemm", l["kind"])]
    assert rc == rec.dsv.OK and l["kind"] == "gemm_nt" and (l["split"], l["pieces"], l["half"]) == (l["tiles"], 2, 0)


@pytest.mark.parametrize("Tt,K,N", [(1007, 5880, 9016), (6498, 840, 8224), (2337, 2424, 8104)])
def test_one_wave_of_dx_is_halved_either_way(rec, Tt, K, N):
    """dX of one partial wave over about 130 K-steps: half tiles with W as it is and transposed,
    which must give the same bits, and no pieces (timed in 163 .. 284 us, halves 141 .. 177)."""
    for wt in (False, True):
        rc, launches = rec.bwd_grouped(rec.plan([(0, Tt, 0, 1)], [16], 16), [(K, N)], wt=wt)
        l, = [l for l in launches if re.match("part|gemm", l["kind"])]
        assert rc == rec.dsv.OK and l["kind"] == ("gemm_nt" if wt else "gemm_nn")
        assert (l["split"], l["half"]) == (0, l["tiles"])


@pytest.mark.parametrize("T", [8192, 8193, 32768, 32769, 70000])
def test_rows_of_the_sum_fit_its_grid(rec, T):
    """Every row with an adapter of its own: the sum has a row of workgroups for each 16 rows of
    an item, at most 65535; more rows than that take tiles."""
    p = rec.plan([(t, 1, t, 1) for t in range(T)], [4] * T, 4)
    for K, N in ((8192, 8), (8192, 64), (64, 8192), (8, 8192), (65536, 64), (64, 65536)):
        for bwd, (rc, launches) in enumerate((rec.fwd(p, K, N), rec.bwd_grouped(p, [(K, N)]))):
            sums = [l for l in launches if l["kind"] == "finish"]
            assert rc == rec.dsv.OK and (not sums or (2 - bwd) * sums[0]["items"] <= 65535), (K, N, launches)
            assert T <= (32768 if bwd else 8192) or not sums, (K, N, launches)


@pytest.mark.parametrize("rank,N,halves", [(64, 512, 0), (64, 4096, 128), (16, 512, 128)])
def test_halves_leave_room_for_wide_side_work(rec, rank, N, halves):
    """Grouped backward of 501 rows through two projections of 8192 columns, 128 tiles: over
    a short contraction they stay whole where the dA reduction of rank 64 runs beside them."""
    p = rec.plan([(0, 501, 0, 1)], [rank], 64)
    rc, launches = rec.bwd_grouped(p, [(8192, N)] * 2)
    if "part" in {l["kind"] for l in launches}:  # the longer contraction runs in pieces where they fit
        rc, launches = rec.bwd_grouped(p, [(8192, N)] * 2, short=256)
    tiles = [l for l in launches if l["kind"] == "group_nt"]
    assert rc == rec.dsv.OK and len(tiles) == 2 and sum(l["half"] for l in tiles) == halves, launches


# What the GPU tests below are named for, at 256 compute units.

def test_gpu_tests_of_split_tiles_reach_them(rec):
    """A workspace 256 bytes short of the pieces: 256 x 256 tiles split along the contraction."""
    import test_gpu_dropout
    import test_gpu_parity
    for m in (test_gpu_parity, test_gpu_dropout):
        p = rec.plan(m.SPLIT, m.SPLIT_RANKS, 64)
        calls = [rec.fwd(p, 4096, 2000, short=256), rec.bwd_grouped(p, [(4096, 2000)], wt=False, short=256)]
        calls += [rec.bwd_grouped(p, [(4096, 2000)], wt=wt, dropout=True, short=256) for wt in (False, True)]
        for i, (rc, launches) in enumerate(calls):
            l, = [l for l in launches if re.match("part|gemm|group", l["kind"])]
            assert rc == rec.dsv.OK and l["tm"] == 256 and l["split"] == l["tiles"] > 0 and l["pieces"] > 1
            assert l["drop"] == (i >= 2) and l["kind"] == ("gemm_nt" if i in (0, 3) else "gemm_nn")


def test_gpu_tests_of_half_tiles_reach_them(rec):
    """Masked dX: the whole and the halved tiles, with W as it is and transposed; the group of
    three that the bits are compared with has whole tiles only."""
    import test_gpu_pieces
    for Tt, K, N, n, whole, halves in test_gpu_pieces.MASKED_HALVES:
        p = rec.plan([(0, 200, 0, 1), (200, Tt - 300, 1, 1), (Tt - 100, 99, 2, 1), (Tt - 1, 1, 0, 1)], [16, 8, 40], 64)
        for wt in (False, True):
            for m, want in ((n, (whole, halves)), (3, (None, 0))):
                if m != n and n == 1:
                    continue
                rc, launches = rec.bwd_grouped(p, [(K, N)] * m, wt=wt, dropout=True)
                tiles = [l for l in launches if re.match("part|gemm|group", l["kind"])]
                assert rc == rec.dsv.OK and all(l["drop"] and l["split"] == 0 for l in tiles)
                assert sum(l["half"] for l in tiles) == want[1], (Tt, m, tiles)
                assert want[0] is None or sum(l["whole"] for l in tiles) == want[0], (Tt, m, tiles)


def test_gpu_tests_of_pieces_reach_every_tile(rec):
    """The pieces' four tiles in each pass."""
    import test_gpu_pieces as tp
    seen = {"fwd": set(), "bwd": set()}
    for T, Tt, K, N, r_max, ranks in tp.CASES:
        p = rec.plan(tp._segments(T, Tt, len(ranks)), ranks, r_max)
        for shapes in ([(K, N)], [(K, N), (K, 2 * N)]):
            seen["fwd"] |= {l["cfg"] for l in rec.fwd_grouped(p, shapes)[1] if l["kind"] == "part"}
            seen["bwd"] |= {l["cfg"] for l in rec.bwd_grouped(p, shapes)[1] if l["kind"] == "part"} if Tt else set()
    for T, tile in tp.WIDE_PIECES.items():
        p = rec.plan([(0, 100, 0, 1), (100, 29, 1, 1), (129, T - 129, 2, 1)], [12, 8, 5], 12)
        for ps, call in (("fwd", rec.fwd_grouped), ("bwd", rec.bwd_grouped)):
            cfg, = {l["cfg"] for l in call(p, [(2056, 2056)] * 2)[1] if l["kind"] == "part"}
            assert cfg == {(128, 128): 2, (128, 256): 3}[tile]
            seen[ps].add(cfg)
    assert seen == {"fwd": {0, 1, 2, 3}, "bwd": {0, 1, 2, 3}}
