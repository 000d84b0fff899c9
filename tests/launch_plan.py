"""What the library launches for a GEMM, asked on the host: csrc/jet_plan.h compiled with g++, no GPU involved."""
from __future__ import annotations

import ctypes
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_14243_amd", "csrc")
CUS = 256

SHIM = """
#include "jet_plan.h"
extern "C" int jet_plan(int row_scales, long I, long J, long G, long cus, int whole, long* out) {
    const jet::GemmPlan p = jet::plan_gemm(row_scales, I, J, G, cus, whole);
    out[0] = p.bm; out[1] = p.bn; out[2] = p.split; out[3] = p.panel;
    out[4] = p.depth; out[5] = p.nt; out[6] = jet::resident_per_cu(p.kernel);
    return p.kernel;
}
extern "C" int jet_quotient(int n, int d) { return jet::quotient(n, d, jet::reciprocal(d)); }
extern "C" void jet_chunk(int lane, int row, int step, int* out) {
    out[0] = jet::chunk_row(lane); out[1] = jet::chunk_step(lane);
    out[2] = jet::chunk_place(row) + ((16 * step) ^ jet::chunk_swap(row));
}
extern "C" int jet_tile(int t, long* out) {
    if (t >= jet::kNumGemmTiles) return -1;
    out[0] = jet::kGemmTiles[t].bm; out[1] = jet::kGemmTiles[t].bn;
    return jet::kGemmTiles[t].kernel;
}
"""
KERNELS = ("strips", "panel", "small", "small deep", "half", "wide", "big", "split rows", "split columns")

_lib = None


def lib():
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
            with open(src, "w") as f:
                f.write(SHIM)
            subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", f"-I{CSRC}", src, "-o", so], check=True)
            _lib = ctypes.CDLL(so)
        _lib.jet_plan.argtypes = [ctypes.c_int] + [ctypes.c_long] * 4 + [ctypes.c_int, ctypes.POINTER(ctypes.c_long)]
    return _lib


def _plan(I, J, R, row_scales=False, cus=CUS, whole=True):
    out = (ctypes.c_long * 7)()
    return KERNELS[lib().jet_plan(row_scales, I, J, R // 128, cus, whole, out)], list(out)


def plan(I: int, J: int, R: int, row_scales: bool = False, **kw):
    """(kernel, rows of the tile, columns of the tile, split) of OUT[I,J] over a reduction of R.  Keywords: cus, whole."""
    k, out = _plan(I, J, R, row_scales, **kw)
    return k, out[0], out[1], out[2]


def strip_depth(I: int, J: int, R: int) -> int:
    """Units in flight per wave, 0 where the launch runs no strips."""
    return _plan(I, J, R)[1][4]


def past_the_caches(I: int, J: int, R: int) -> bool:
    """Whether the decode kernel reads its weights with the policy of lines that are not needed again."""
    return bool(_plan(I, J, R)[1][5])


def launches(I: int, J: int, R: int, row_scales: bool = False, whole: bool = True):
    """Launches of a GEMM on the tile kernel: (kernel and tile, tiles of the workgroup that has most)."""
    k, (bm, bn, split, _, _, _, per_cu) = _plan(I, J, R, row_scales=row_scales, whole=whole)
    if k.startswith("split"):
        rows = k == "split rows"
        parts = ((split, J), (I - split, J)) if rows else ((I, split), (I, J - split))
        return [launch for i, j in parts for launch in launches(i, j, R, row_scales, whole=False)]
    n_tiles = -(-I // bm) * -(-J // bn)
    return [(f"{k} {bm}x{bn}", -(-n_tiles // min(n_tiles, CUS * per_cu)))]


def name(I: int, J: int, R: int, **kw) -> str:
    """"strips", or kernel and tile: "panel 32x16", "big 256x256", "split rows 256x256"."""
    k, bm, bn, _ = plan(I, J, R, **kw)
    return k if k == "strips" else f"{k} {bm}x{bn}"


def chunk(lane: int = 0, row: int = 0, step: int = 0):
    """(row, step) that a lane of a scale copy brings, and the byte of a row's step in the chunk."""
    out = (ctypes.c_int * 3)()
    lib().jet_chunk(lane, row, step, out)
    return (out[0], out[1]), out[2]


def tiles():
    out, t = (ctypes.c_long * 2)(), 0
    while (k := lib().jet_tile(t, out)) >= 0:
        yield f"{KERNELS[k]} {out[0]}x{out[1]}"
        t += 1
