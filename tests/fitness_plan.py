"""The plan of a float32 fitness launch and the route of a small run as the
library chooses them (host code, no GPU needed), for tests whose shapes have to
reach a certain kernel."""
import ctypes
from collections import namedtuple

from paper_1304_0597_amd import game

Plan = namedtuple("Plan", "cols tiles_per_split splits last_split chunks")


class _Draw(ctypes.Structure):
    _fields_ = [("seed", ctypes.c_uint64), ("thr_mut", ctypes.c_uint64), ("sigma", ctypes.c_float)] + \
        [(n, ctypes.c_int32) for n in ("K", "E", "P", "n_pairs", "blocks")] + \
        [(n, ctypes.c_void_p) for n in ("words", "mut", "cur")] + [("n_items", ctypes.c_int32)]


class _Fit(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("X", "t", "genes", "genes_alt", "gen_sel", "stop",
                                               "stop_seen", "gen_seen", "partial")] + \
        [("NP", ctypes.c_int64)] + \
        [(n, ctypes.c_int32) for n in ("N", "K", "n_chrom", "U", "Q", "pairs_per_chunk", "n_chunks",
                                       "n_ctiles", "ld_partial", "n_splits", "tiles_per_split",
                                       "n_tiles", "xcd_remap", "error_fn")] + \
        [("R", ctypes.c_float), ("degree", ctypes.c_int32), ("basis", ctypes.c_int32),
         ("cs", ctypes.c_void_p), ("tile_cols", ctypes.c_int32), ("draw", _Draw)]


class _GA(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("pop_a", "pop_b", "out_a", "out_b", "fitness", "order",
                                               "gen_ptr", "stop")] + \
        [(n, ctypes.c_int32) for n in ("generation", "P", "K", "k", "E", "elite_mode")] + \
        [("thr_cross", ctypes.c_uint64), ("thr_mut", ctypes.c_uint64), ("sigma", ctypes.c_float),
         ("seed", ctypes.c_uint64), ("n_slots", ctypes.c_int32), ("children", ctypes.c_void_p),
         ("selection", ctypes.c_int32), ("cum", ctypes.c_void_p)]


def _planned(NP, N, d, P, basis, error_fn=0):
    """FitArgs (csrc/common.h) as plan_fitness leaves them."""
    fn = game.lib()["_ZN4game12plan_fitnessERNS_7FitArgsEiib"]
    fn.argtypes = [ctypes.POINTER(_Fit), ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    fn.restype = None
    a = _Fit(NP=NP, N=N, n_chrom=P, degree=d, basis=basis, error_fn=error_fn)
    fn(ctypes.byref(a), d, basis, True)
    assert a.NP == NP and a.n_splits == -(-a.n_tiles // a.tiles_per_split)
    return a


def plan(NP, N, d, P, basis=0):
    """Plan for P chromosomes over NP patterns of N features at degree d."""
    a = _planned(NP, N, d, P, basis)
    return Plan(a.tile_cols, a.tiles_per_split, a.n_splits,
                a.n_tiles - a.tiles_per_split * (a.n_splits - 1), a.n_chunks)


def resident(NP, N, d, P, basis=0, error_fn=0, selection=0, tournament_k=4, elitism=2, elite_mode=0):
    """Whether such a run takes the one-workgroup kernel."""
    f = _planned(NP, N, d, P, basis, error_fn)
    f.cs = 1 if basis == 3 else None      # a table there is: only tested for null
    g = _GA(P=P, K=(2 if basis == 3 else 1) * N * d + 1, k=tournament_k, E=elitism,
            elite_mode=elite_mode, selection=selection)
    fn = game.lib()["_ZN4game13resident_fitsERKNS_7FitArgsERKNS_6GAArgsE"]
    fn.argtypes = [ctypes.POINTER(_Fit), ctypes.POINTER(_GA)]
    fn.restype = ctypes.c_bool
    return bool(fn(ctypes.byref(f), ctypes.byref(g)))


# Shapes (NP, N, d, P) that reach a kernel or a branch of one, with the columns and
# tiles per split, the last split's tiles and the gene chunks of their plans.
REACHES = {
    # 64-chromosome tiles: general rows, narrow rows by single features and by quads,
    # one tile and more than one to a split
    "64-general-1": ((100001, 20, 3, 40), (64, 1, 1, 1)),
    "64-general-2": ((200001, 20, 1, 33), (64, 2, 2, 1)),
    "64-general-quads-2": ((200001, 12, 4, 40), (64, 2, 2, 1)),
    "64-narrow-quads-1": ((90001, 8, 1, 40), (64, 1, 1, 1)),
    "64-narrow-quads-2": ((200001, 8, 1, 40), (64, 2, 2, 1)),
    "64-narrow-rows-1": ((100001, 5, 3, 50), (64, 1, 1, 1)),
    "64-narrow-rows-2": ((200001, 7, 4, 50), (64, 2, 2, 1)),
    # 128-chromosome tiles: gene chunks over splits of 3 and of 4 tiles whose last one
    # has 1 and 3 (a wave group without a tile joins the chunk barriers), whole genes
    # over odd splits, an odd last feature pair at degree 4
    "128-chunks-3-last-1": ((20000, 40, 9, 900), (128, 3, 1, 3)),
    "128-chunks-4-last-3": ((100000, 40, 9, 256), (128, 4, 3, 3)),
    "128-odd-5-last-2": ((40001, 9, 4, 1000), (128, 5, 2, 1)),
    "128-pairs-of-quads-3": ((20001, 40, 2, 900), (128, 3, 1, 1)),
    # 32-chromosome tiles, narrow rows over several tiles to a split: the next tile
    # read ahead, quads and single features
    "32-narrow-quads-2": ((300001, 16, 1, 23), (32, 2, 2, 1)),
    "32-narrow-rows-2": ((300001, 15, 1, 23), (32, 2, 2, 1)),
    "32-narrow-rows-5": ((600001, 7, 4, 20), (32, 5, 4, 1)),
    "32-narrow-quads-d3": ((400001, 8, 3, 20), (32, 2, 1, 1)),
}


def reached(name, basis=0):
    """The shape, after a check that its plan is still the one that it is for."""
    shape, want = REACHES[name]
    p = plan(*shape, basis)
    chunks = 2 * want[3] if basis == 3 and want[3] > 1 else want[3]    # twice the terms
    assert (p.cols, p.tiles_per_split, p.last_split, p.chunks) == (*want[:3], chunks), (name, p)
    return shape
