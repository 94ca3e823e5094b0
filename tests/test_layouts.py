"""Launch shapes that the library plans on the host (tile width, split counts, slabs, scratch), for sizes
from one water to 128, through a small program linked against the library (no GPU)."""
import os
import subprocess

import pytest

N = pytest.importorskip("paper_2404_09452_amd._native")
if not os.path.exists(N.LIB_PATH):
    pytest.skip("libdfjk.so not built", allow_module_level=True)
from paper_2404_09452_amd import build as B  # noqa: E402
from paper_2404_09452_amd import dfjk as G  # noqa: E402

FP64, FP32, BF16X3, INT8, INT8_FAST = range(5)
CUS = 256          # compute units a plan assumes
T = 128            # tile of the increment
WATERS = (1, 2, 3, 5, 7, 10, 12, 16, 20, 24, 25, 28, 31, 32, 35, 37, 44, 48, 55, 64, 96, 128)


@pytest.fixture(scope="module")
def query(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("layout") / "layout_query")
    here = os.path.dirname(os.path.abspath(__file__))
    lib = os.path.dirname(N.LIB_PATH)
    cmd = [B.HIPCC] + B.FLAGS + [os.path.join(here, "layout_query.cpp"), "-L" + lib,
                                 "-l:" + os.path.basename(N.LIB_PATH), "-Wl,-rpath," + lib, "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True)

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, check=True)
        return [[int(x) for x in line.split()] for line in r.stdout.splitlines()]
    return ask


def sizes(n, extra=0):
    """nao, naux_pad and nf_pad (every pair kept) of n waters in the test basis, with more s functions."""
    nao = 30 * n + extra
    return nao, -(-87 * n // 128) * 128, -(-nao * (nao + 1) // 2 // 64) * 64


class Layout:
    def __init__(self, v):
        self.ktile, self.nsplit, self.nsub, self.slab, self.nslab, self.kdim, self.bytes, self.kpart = v


def layouts(query, asked):
    """asked: dicts with n, nocc, precision and any of the options below."""
    lines = []
    for a in asked:
        o = dict(aux_slab=0, k_tile=0, tuned=(0, 0), with_D=0, delta=0, nsplit=0, overlap=1, force_slab=0, ktile=0)
        o.update(a)
        nao, naux, nf = sizes(o["n"], o.get("extra", 0))
        lines.append("layout %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d" % (
            nao, naux, nf, o["aux_slab"], o["k_tile"], *o["tuned"], o["nocc"], o["precision"], o["with_D"], o["delta"],
            o["nsplit"], o["overlap"], o["force_slab"], o["ktile"]))
    return [Layout(v) for v in query(lines)]


@pytest.mark.parametrize("precision", [FP64, FP32])
def test_increment_splits(query, precision):
    """The increment's reduction reads both triangles of every split, one of them across rows, so an extra
    split costs it more than it gives the product: no more splits than one per 256 k (FP64) and than fill the
    chip twice (FP32), and no parts."""
    for n in WATERS:
        L, = layouts(query, [dict(n=n, nocc=5 * n, precision=precision, delta=1)])
        tiles = (-(-30 * n // T)) ** 2
        assert L.ktile == T and L.nsub == 1
        assert L.nsplit <= max(1, L.kdim // 256)
        assert L.nsplit <= max(1, (16 if precision == FP64 else 2) * CUS // tiles)


@pytest.mark.parametrize("precision", [FP64, FP32, BF16X3, INT8, INT8_FAST])
def test_autotune_candidates(query, precision):
    """Every candidate of the autotuner survives its code (1000 tile + splits), is the shape that its own
    layout has, and leaves the ranges of the FP32 folds where they are; the built-in shape is among them."""
    for n in WATERS:
        for nocc in (1, 5 * n, 30 * n):
            nao, naux, nf = sizes(n)
            row, = query(["candidates %d %d %d 0 0 0 0 %d %d" % (nao, naux, nf, nocc, precision)])
            cands = list(zip(row[::2], row[1::2]))
            assert len(cands) <= 16 and len(set(cands)) == len(cands)
            built = layouts(query, [dict(n=n, nocc=nocc, precision=precision, nsplit=-1)])[0]
            assert (built.ktile, built.nsplit) in cands
            own = layouts(query, [dict(n=n, nocc=nocc, precision=precision, nsplit=s, ktile=t) for t, s in cands])
            for (t, s), L in zip(cands, own):
                assert s > 0 and G.k_shape(1000 * t + s) == (t, s)
                assert (L.ktile, L.nsplit) == (t, s)
                assert L.nsplit // L.nsub == built.nsplit // built.nsub or precision != FP32


@pytest.mark.parametrize("precision", [FP64, FP32, BF16X3, INT8, INT8_FAST])
def test_static_build_after_autotuning(query, precision):
    """A build that fits the 64 MiB static scratch untuned also fits it whichever candidate the autotuner
    keeps, on that candidate's tile where the tuned shape fits and as untuned otherwise."""
    fitted = 0
    for n in range(1, 15):
        for nocc in (1, 5 * n, 15 * n):
            size = "%d %d %d" % sizes(n)
            row, = query(["candidates %s 0 0 0 0 %d %d" % (size, nocc, precision)])
            shapes = [(0, 0)] + list(zip(row[::2], row[1::2]))
            got = query(["static %s 0 0 %d %d %d %d" % (size, t, s, nocc, precision) for t, s in shapes])
            if not got[0][0]:
                continue
            fitted += 1
            for (t, s), g in zip(shapes, got):
                assert g[0] == 1 and g[4] <= 64 << 20, (n, nocc, t, s)
                assert s == 0 or g[1] == t or g == got[0]
    assert fitted >= 20


def test_fp32_parts_are_not_empty(query):
    """No part of an FP32 k range is empty: built-in splits and the autotuner's, one slab and several."""
    for n in WATERS:
        for nocc, slab in ((1, 0), (5 * n, 0), (30 * n, 0), (5 * n, 128), (5 * n, 640)):
            nao, naux, nf = sizes(n)
            row, = query(["candidates %d %d %d %d 0 0 0 %d %d" % (nao, naux, nf, slab, nocc, FP32)])
            asked = [(0, -1)] + list(zip(row[::2], row[1::2]))
            for L in layouts(query, [dict(n=n, nocc=nocc, precision=FP32, aux_slab=slab, nsplit=s, ktile=t)
                                     for t, s in asked]):
                ranges = L.nsplit // L.nsub
                part = -(-(-(-L.kdim // ranges)) // L.nsub)       # k of a part ...
                part = -(-part // 512) * 512 if L.nsub > 1 else part   # ... in whole folds
                assert ranges * L.nsub == L.nsplit
                assert (L.nsub - 1) * part < -(-L.kdim // ranges)


def test_fp32_partials_stay_small(query):
    """FP32 parts do not multiply the partial tiles of many aux slabs: within 6 GB wherever whole ranges (one
    round of two 128-wide workgroups a CU for every slab) are."""
    for n in WATERS:
        for slab in (0, 128, 256, 640, 1024):
            L, = layouts(query, [dict(n=n, nocc=5 * n, precision=FP32, aux_slab=slab)])
            assert L.kpart <= max(6e9, L.kpart // L.nsub), (n, slab)


# whole FP64 builds, time on 64-wide over time on 96-wide tiles (AO count: n waters and more s functions)
MEASURED = {(16, 32): 0.872, (18, 0): 0.938, (19, 6): 0.946, (20, 0): 0.886, (21, 0): 0.899, (23, 0): 0.889,
            (24, 0): 0.932, (24, 16): 0.964, (25, 0): 0.971, (25, 18): 0.977, (26, 0): 0.898, (27, 0): 0.935,
            (28, 24): 1.033, (29, 0): 0.908, (30, 0): 0.986, (31, 0): 0.992, (32, 0): 1.014, (32, 16): 0.958,
            (33, 0): 0.977, (33, 18): 0.974, (35, 0): 1.070, (35, 6): 1.075, (36, 0): 0.957, (37, 0): 1.041,
            (38, 12): 1.041, (39, 0): 1.011, (40, 0): 0.991, (42, 0): 0.992, (44, 24): 1.044, (47, 0): 1.119}


def test_fp64_tile_width_follows_measurement(query):
    """The FP64 tile rule takes the width that was faster wherever the two differ by 1% or more (1.5% on the
    side of 96-wide tiles, whose ragged sizes it takes as 64-wide)."""
    for (n, extra), ratio in MEASURED.items():
        L, = layouts(query, [dict(n=n, extra=extra, nocc=5 * n, precision=FP64)])
        if ratio <= 0.99:
            assert L.ktile == 64, 30 * n + extra
        elif ratio >= 1.015:
            assert L.ktile == 96, 30 * n + extra
    assert layouts(query, [dict(n=32, nocc=160, precision=FP64)])[0].ktile == 96
