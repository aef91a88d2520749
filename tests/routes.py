"""The library's choice of kernel for a matrix-core linear or for the fused decode
attention, asked on the host (no GPU): the C++ functions behind the entry
points, by their mangled names."""
import ctypes

from paper_2605_08755_amd import laq

# MfmaRoute of csrc/laq_internal.h, in order.
NAMES = ("stream", "share", "quad_wave", "quad_wave_regs", "quad_wave_codes", "walk4", "walk8", "split_stream", "split",
         "one_tile_codes", "two_tiles")


class StreamPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in "MT PH D nb TS nq W nblocks ranges".split()] + [("lds", ctypes.c_uint32)]


class SplitPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("S", "qs", "tile_blocks")]


def _bind(name, restype, *argtypes):
    f = getattr(laq.lib(), name)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def route(bits, M, N, K, workspace=False):
    """Name of the kernel that takes the call; workspace: with split-K scratch."""
    i, l = ctypes.c_int, ctypes.c_int64
    return NAMES[_bind("_ZN3laq10mfma_routeEiillb", i, i, i, l, l, ctypes.c_bool)(bits, M, N, K, workspace)]


def stream_plan(bits, M, N, G, ranges):
    i = ctypes.c_int
    return _bind("_ZN3laq11stream_planEiilii", StreamPlan, i, i, ctypes.c_int64, i, i)(bits, M, N, G, ranges)


def split_plan(M, N, G):
    i = ctypes.c_int
    return _bind("_ZN3laq15mfma_split_planEili", SplitPlan, i, ctypes.c_int64, i)(M, N, G)


def group_quad_wave(M, tiles, nq):
    """Form of the one-wave-per-quad kernel that a group takes (0 up-front, 1 in
    64 registers), or -1: the kernel whose waves walk several quads."""
    i = ctypes.c_int
    return _bind("_ZN3laq20mfma_group_quad_waveEili", i, i, ctypes.c_int64, i)(M, tiles, nq)


def attention_long(Hq, Hkv, pos):
    """Whether the fused attention runs in the long-context kernel."""
    l = ctypes.c_int64
    return _bind("_ZN3laq22attention_long_contextElll", ctypes.c_bool, l, l, l)(Hq, Hkv, pos)
