"""The library's rules on sizes (csrc/mq_plan.h) for tests that have to know which form a call takes: built with the host
compiler on first use, no GPU needed."""
import ctypes
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_06786_amd", "csrc")

SOURCE = r'''
#include "mq_plan.h"
using namespace mq;
extern "C" void plan_forward(int64_t M, int64_t N, int64_t K, int nr, int64_t *out) {
    const FwdSplitPlan p = make_split_plan(M, N, K, nr);
    int tiled = 0;
    fwd_tiled_cost(M, N, K, nr, &tiled);
    out[0] = p.mb, out[1] = p.splits, out[2] = nr == 1 ? fwd_wide_mb(M, N, K, nullptr) : 0, out[3] = tiled;
}
extern "C" int plan_loss_arrivals(void) { return (int)kLossArrivals; }
extern "C" void plan_dx(int64_t M, int64_t N, int64_t K, int nr, int64_t *out) {
    const DxPlan p = make_dx_plan(M, N, K, nr);
    out[0] = p.mb, out[1] = p.splits;
}
extern "C" void plan_dw(int64_t M, int64_t N, int64_t K, int batch, int64_t *out) {
    const DwPlan p = make_dw_plan(M, N, K, batch);
    out[0] = p.hb, out[1] = p.whole, out[2] = p.rest, out[3] = p.parts;
}
extern "C" int plan_dw_turns(int64_t M, int64_t N, int64_t K, int batch, int alone, int prep) {
    return dw_turns(M, N, K, batch, alone, prep, make_dw_plan(M, N, K, batch).hb);
}
extern "C" int plan_dw_first(int64_t M, int64_t N, int64_t K) { return dw_first(M, N, K); }
extern "C" int plan_dw_in_place(int64_t M, int64_t N, int64_t K, int64_t X, int64_t dY, int64_t dX, int64_t dW) {
    return dw_turns_in_place(M, N, K, (const void *)X, (const void *)dY, (const void *)dX, (const void *)dW, true, make_dw_plan(M, N, K, 1).hb);
}
extern "C" void plan_quad(int64_t B, int64_t N, int64_t K, int r, int list, int64_t *out) {
    const QuadPlan p = make_quad_plan(B, N, K, K * r / 8, r, list);
    out[0] = p.depth > 0 ? p.ks * p.rw : 0, out[1] = p.nl, out[2] = p.list_waves, out[3] = p.shared;
}
extern "C" void plan_gemv(int64_t B, int64_t N, int64_t K, int r, int64_t *out) {
    const GemvPlan p = make_gemv_plan(B, N, K * r / 8, r);
    out[0] = p.rg, out[1] = gemv_roomy(r, p.rg) ? (p.tight ? 128 : 256) : 0, out[2] = p.ngroups, out[3] = p.lds;
}
extern "C" void plan_gemv_split(int64_t B, int64_t N, int64_t K, int r, int64_t *out) {
    const GemvSplitPlan p = make_gemv_split_plan(B, N, K * r / 8, r);
    out[0] = p.groups, out[1] = p.nl, out[2] = p.depth, out[3] = p.ch;
}
'''

# form: "split" (K cut into `ranges`), "wide" (256-channel tiles), "tiled"; blocks: tile height in blocks of 32 tokens
Forward = namedtuple("Forward", "form blocks ranges")
Dx = namedtuple("Dx", "blocks ranges")              # ranges: of channels
Dw = namedtuple("Dw", "side whole cut ranges")      # tiles of side x side: run whole, cut into `ranges` of tokens each
# decode, up to four sequences on tall planes: waves that stream the plane (0: another form), lines per slice, waves for the list, whether
# the former help with it
Quad = namedtuple("Quad", "waves lines list_waves shared")
# decode, general form: 16-row groups per wave, registers the kernel is held to (0: it needs no more than 128), workgroups' worth of rows, LDS
Gemv = namedtuple("Gemv", "row_groups registers groups lds")
# decode with K split: groups of four slices of `lines` lines, ring of `depth` tiles per wave (0: the form does not fit), row blocks per wave
GemvSplit = namedtuple("GemvSplit", "groups lines depth blocks")


@functools.lru_cache(maxsize=None)
def _lib():
    folder = tempfile.mkdtemp(prefix="mq_plans_")
    src, so = os.path.join(folder, "plans.cpp"), os.path.join(folder, "plans.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    for f in (lib.plan_forward, lib.plan_dx, lib.plan_dw, lib.plan_gemv, lib.plan_gemv_split):
        f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int, ctypes.POINTER(ctypes.c_int64)]
        f.restype = None
    lib.plan_dw_in_place.argtypes = [ctypes.c_int64] * 7
    lib.plan_dw_first.argtypes = [ctypes.c_int64] * 3
    lib.plan_dw_turns.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 3
    lib.plan_quad.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 2 + [ctypes.POINTER(ctypes.c_int64)]
    lib.plan_quad.restype = None
    return lib


def _ask(name, *sizes):
    out = (ctypes.c_int64 * 4)()
    getattr(_lib(), name)(*sizes, out)
    return list(out)


def forward(M, N, K, nr, objective=False):
    mb, splits, wide, tiled = _ask("plan_forward", M, N, K, nr)
    if mb:
        return Forward("split", mb, splits)
    return Forward("wide", wide, 1) if wide and not objective else Forward("tiled", tiled, 1)


def loss_workgroups(M, N, K, nr):
    """Form and workgroups of the kernel that leaves the sums of a forward with the objective."""
    form, blocks, _ = forward(M, N, K, nr, objective=True)
    tiles = -(-M // (32 * blocks)) * -(-N // 128)
    return form, 4 * blocks * tiles if form == "split" else tiles


def loss_arrivals():
    """Most workgroups among which the last one to arrive finishes the losses."""
    return _lib().plan_loss_arrivals()


def dx(M, N, K, nr):
    return Dx(*_ask("plan_dx", M, N, K, nr)[:2])


def dw(M, N, K, gradients=1):
    hb, whole, rest, parts = _ask("plan_dw", M, N, K, gradients)
    return Dw(64 * hb, whole, rest, parts)


def dw_turns(M, N, K, gradients=1, alone=True, prep=True):
    """Whether dW takes its operands as they stand; alone: gradients neither summed nor scaled, prep: a preparation runs anyhow."""
    return bool(_lib().plan_dw_turns(M, N, K, gradients, alone, prep))


def dw_first(M, N, K):
    """Whether a backward from copies forms dW before dX."""
    return bool(_lib().plan_dw_first(M, N, K))


def dw_in_place(M, N, K, X, dY, dX, dW):
    """Whether the dW of a backward with a preparation reads its operands as they stand; addresses, dY None where the gradient is summed or scaled,
    dX None where it is not wanted."""
    return bool(_lib().plan_dw_in_place(M, N, K, X, dY or 0, dX or 0, dW))


def quad(B, N, K, r, with_list=False):
    waves, lines, list_waves, shared = _ask("plan_quad", B, N, K, r, int(with_list))
    return Quad(waves, lines, list_waves, bool(shared))


def gemv(B, N, K, r):
    return Gemv(*_ask("plan_gemv", B, N, K, r))


def gemv_split(B, N, K, r):
    return GemvSplit(*_ask("plan_gemv_split", B, N, K, r))
