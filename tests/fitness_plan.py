"""The plan of a float32 fitness launch as the library makes it (host code, no
GPU needed), for tests whose shapes have to reach a certain kernel."""
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


def plan(NP, N, d, P, basis=0):
    """Plan for P chromosomes over NP patterns of N features at degree d
    (FitArgs and plan_fitness of csrc/common.h)."""
    fn = game.lib()["_ZN4game12plan_fitnessERNS_7FitArgsEiib"]
    fn.argtypes = [ctypes.POINTER(_Fit), ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    fn.restype = None
    a = _Fit(NP=NP, N=N, n_chrom=P, degree=d, basis=basis)
    fn(ctypes.byref(a), d, basis, True)
    assert a.NP == NP and a.n_splits == -(-a.n_tiles // a.tiles_per_split)
    return Plan(a.tile_cols, a.tiles_per_split, a.n_splits,
                a.n_tiles - a.tiles_per_split * (a.n_splits - 1), a.n_chunks)
