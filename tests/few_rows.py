"""Calls that reach every launch shape of the few-row kernel (csrc/ccq_few.hip), and the rule's own answer to which one a call takes."""
import ctypes

import numpy as np

from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

FORMATS = {"narrow": [b.NARROW], "wide": [b.WIDE], "mixed": [b.NARROW, b.WIDE], "h16": b.H16}

# (format, (16-row tiles of a pass, row tiles of a wavefront, wavefronts side by side, shares of K), K, N, experts, rows of the
# first expert, every which expert has rows, host offsets given)
CASES = [
    ("narrow", (1, 1, 2, 1), 320, 608, 64, 5, 1, True),
    ("narrow", (1, 1, 2, 2), 320, 17, 4, 5, 1, True),
    ("narrow", (1, 1, 2, 4), 576, 17, 2, 5, 1, True),
    ("narrow", (1, 1, 4, 1), 128, 17, 4, 5, 1, True),
    ("narrow", (1, 1, 4, 2), 320, 196, 48, 16, 8, False),
    ("narrow", (1, 1, 4, 4), 960, 219, 128, 5, 8, False),
    ("narrow", (1, 2, 4, 1), 128, 1454, 48, 5, 1, False),
    ("narrow", (1, 2, 4, 2), 896, 290, 64, 5, 1, True),
    ("narrow", (1, 2, 8, 1), 128, 1849, 32, 5, 1, False),
    ("narrow", (2, 1, 2, 1), 192, 1047, 32, 20, 1, True),
    ("narrow", (2, 1, 2, 2), 320, 20, 1, 20, 1, False),
    ("narrow", (2, 1, 2, 4), 576, 17, 2, 20, 1, False),
    ("narrow", (2, 1, 4, 1), 128, 18, 1, 16, 1, False),
    ("narrow", (2, 1, 4, 2), 320, 19, 1, 32, 1, True),
    ("narrow", (2, 2, 4, 1), 128, 687, 128, 20, 1, True),
    ("narrow", (2, 2, 4, 2), 320, 396, 48, 16, 1, False),
    ("narrow", (2, 2, 8, 1), 128, 762, 48, 20, 1, False),
    ("wide", (1, 1, 2, 1), 128, 785, 48, 5, 1, True),
    ("wide", (1, 1, 2, 2), 576, 20, 3, 5, 1, True),
    ("wide", (1, 1, 2, 4), 1280, 18, 3, 5, 1, True),
    ("wide", (1, 1, 4, 1), 128, 17, 2, 5, 1, False),
    ("wide", (1, 1, 4, 2), 896, 80, 128, 16, 8, False),
    ("wide", (1, 1, 4, 4), 1280, 221, 128, 5, 8, False),
    ("wide", (1, 2, 4, 1), 128, 672, 128, 5, 1, False),
    ("wide", (1, 2, 4, 2), 640, 406, 48, 5, 1, True),
    ("wide", (2, 1, 2, 2), 640, 21, 1, 16, 1, False),
    ("wide", (2, 1, 4, 1), 128, 18, 1, 16, 1, False),
    ("wide", (2, 1, 4, 2), 576, 23, 1, 20, 1, True),
    ("wide", (2, 2, 4, 1), 128, 1043, 64, 16, 1, False),
    ("wide", (2, 2, 4, 2), 704, 173, 128, 16, 1, False),
    ("wide", (2, 2, 8, 1), 128, 316, 128, 20, 1, True),
    ("mixed", (1, 1, 2, 1), 256, 287, 128, 5, 1, True),
    ("mixed", (1, 1, 2, 2), 1216, 18, 2, 5, 1, False),
    ("mixed", (1, 1, 2, 4), 2368, 19, 1, 5, 1, False),
    ("mixed", (1, 1, 4, 1), 128, 17, 3, 5, 1, True),
    ("mixed", (1, 1, 4, 2), 1408, 108, 64, 5, 8, False),
    ("mixed", (1, 2, 4, 1), 128, 473, 128, 5, 1, True),
    ("mixed", (1, 2, 4, 2), 1792, 363, 64, 5, 1, False),
    ("mixed", (2, 1, 2, 2), 1344, 17, 2, 32, 1, True),
    ("mixed", (2, 1, 4, 1), 128, 23, 1, 20, 1, True),
    ("mixed", (2, 1, 4, 2), 1216, 25, 1, 20, 1, True),
    ("mixed", (2, 2, 8, 1), 128, 263, 128, 20, 1, True),
    ("h16", (1, 1, 2, 1), 128, 1602, 24, 5, 1, True),
    ("h16", (1, 1, 2, 2), 576, 19, 2, 5, 1, True),
    ("h16", (1, 1, 2, 4), 1152, 19, 4, 5, 1, False),
    ("h16", (1, 1, 4, 1), 128, 18, 4, 5, 1, False),
    ("h16", (1, 1, 4, 2), 640, 119, 128, 20, 8, False),
    ("h16", (1, 1, 4, 4), 1088, 197, 128, 5, 8, False),
    ("h16", (1, 2, 4, 1), 128, 667, 128, 5, 1, True),
    ("h16", (1, 2, 4, 2), 704, 465, 64, 5, 1, True),
    ("h16", (2, 1, 2, 2), 576, 19, 1, 32, 1, False),
    ("h16", (2, 1, 4, 1), 128, 17, 1, 32, 1, False),
    ("h16", (2, 1, 4, 2), 640, 17, 1, 20, 1, True),
    ("h16", (2, 2, 4, 1), 128, 1116, 64, 16, 1, False),
    ("h16", (2, 2, 4, 2), 576, 304, 64, 20, 1, True),
    ("h16", (2, 2, 8, 1), 128, 283, 128, 20, 1, True),
]

# dense calls on both sides of the lines: (format, K, N, rows, taken)
DENSE = [
    ("narrow", 3072, 300, 16, True), ("narrow", 3136, 300, 16, False), ("narrow", 1536, 40, 17, True), ("narrow", 1600, 40, 17, False),
    ("narrow", 3072, 2040, 32, True), ("narrow", 3136, 2040, 32, False), ("narrow", 3136, 12600, 20, True),
    ("wide", 2048, 100, 16, True), ("wide", 2112, 100, 16, False), ("wide", 3584, 40, 17, True), ("wide", 3648, 40, 17, False), ("wide", 3648, 5840, 20, True),
    ("mixed", 9984, 40, 32, True), ("mixed", 10048, 40, 17, False), ("mixed", 1024, 40, 16, False),
    ("h16", 2048, 100, 5, True), ("h16", 2112, 100, 5, False), ("h16", 4096, 40, 17, True), ("h16", 4160, 40, 32, False), ("h16", 4160, 5600, 20, True),
]


def group_map(family, K):
    G = K // 64
    return synth.group_format_map(G, max(1, G // 3), synth.rng(1, K)) if family == "mixed" else None


def counts(E, top, step):
    return [top] + [(5 * e + 3) % (top + 1) if e % step == 0 else 0 for e in range(1, E)]


def offsets(rows):
    return np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)


def _shape(family, K, N, E, rows, offs):
    f = b.load().ccq_few_launch_shape
    gf = group_map(family, K)   # (the descriptor points into it)
    w = b.descriptor(K, N, FORMATS[family], gf)
    out = np.zeros(5, np.int32)
    assert f(ctypes.byref(w), E, rows, None if offs is None else offs.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p)) == 0
    return out.tolist()


def grouped_shape(family, K, N, rows, host):
    offs = offsets(rows)
    return tuple(_shape(family, K, N, len(rows), int(offs[-1]), offs if host else None)[:4])


def dense_shape(family, K, N, M):
    """The shape, and whether the call takes the kernel at all."""
    s = _shape(family, K, N, 0, M, None)
    return tuple(s[:4]), bool(s[4])
