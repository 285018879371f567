"""Glue used by the tests: oracle results <-> the arrays the library's binding takes."""
import dataclasses
import functools

import numpy as np

from oracle import encoder as oenc
from oracle import gf2
from synth_inputs import CONFIGS, make_workload


# (planes, m, n, columns, blocks of columns and waves of a workgroup, workgroups per tile): layers on 32-row tiles whose
# reduction is cut into two or three parts
CUTS_IN_PARTS = [
    (1, 3000, 7000, 32, 1, 12, 2), (1, 1500, 4100, 64, 1, 8, 2), (1, 3000, 4100, 64, 2, 8, 2), (1, 257, 4100, 8, 1, 8, 3),
    (1, 257, 3600, 64, 1, 8, 3), (1, 2049, 4100, 64, 2, 8, 3), (2, 3000, 3600, 8, 1, 8, 2), (2, 3000, 4100, 32, 1, 12, 2),
    (2, 1500, 3000, 64, 1, 8, 2), (2, 3000, 4100, 64, 2, 8, 2), (2, 257, 2500, 32, 1, 8, 3), (2, 2049, 4100, 64, 2, 8, 3),
    (3, 1500, 1800, 8, 1, 8, 2), (3, 3000, 2500, 32, 1, 8, 2), (3, 257, 2100, 32, 1, 8, 3),
]

# (planes, m, n, n_in, word pairs per wave, rounds): layers on which waves of the few-column kernel end inside a group of word
# pairs whose patch flips are scattered together
FEW_COLUMNS_IN_ROUNDS = [
    (1, 4352, 8448, 8, 5, 2), (1, 8500, 5300, 32, 3, 3), (1, 9216, 5632, 24, 3, 3), (2, 8448, 4352, 8, 3, 3),
    (2, 8500, 4300, 16, 3, 3), (2, 9216, 4608, 24, 3, 3), (3, 6000, 3000, 17, 3, 1), (3, 6000, 3000, 24, 3, 1),
    (3, 9216, 4608, 32, 3, 3), (4, 6000, 3000, 8, 2, 2), (2, 4096, 9216, 16, 5, 1),
]


def paper_format_arrays(enc: "oenc.Encoded"):
    """Oracle `Encoded` -> (w_c uint32[q,l], keep uint64[m*spr] row-major 64-bit words, n_patch uint16[q,l],
    d_patch uint8[], M_rows uint32[n_out])."""
    w_c = gf2.bits_to_int(enc.w_c).astype(np.uint32)
    keep = gf2.bits_to_int(enc.keep.reshape(-1, 64)).astype(np.uint64)
    n_patch = enc.n_patch.astype(np.uint16)
    d_patch = np.concatenate([np.asarray(d, dtype=np.uint8) for d in enc.d_patch]) if enc.q else np.zeros(0, np.uint8)
    M_rows = gf2.bits_to_int(enc.M).astype(np.uint32)
    return w_c, keep, n_patch, d_patch, M_rows


def pack_encoded(enc: "oenc.Encoded"):
    import paper_1905_10138_amd as xe
    w_c, keep, n_patch, d_patch, M_rows = paper_format_arrays(enc)
    return xe.pack(enc.m, enc.n, enc.n_in, enc.q, w_c, keep, n_patch, d_patch, enc.alpha, M_rows, enc.n_out)


@functools.lru_cache(maxsize=8)
def encoded_workload(name: str, m=None, n=None, S=None, n_out=None, n_in=None, exhaustive=False):
    """(workload, oracle-encoded) for a config, cached for the test session.  `S` overrides the
    pruning rate (a low rate with a small n_in gives many patches per slice); `n_out` / `n_in`
    override the slice geometry (the paper's best ratios are at n_out near 200 with n_in = 20);
    `exhaustive` encodes with the 2^n_in search of Section 5.2 in place of Algorithm 1."""
    cfg = CONFIGS[name]
    over = {k: v for k, v in (("S", S), ("n_out", n_out), ("n_in", n_in)) if v is not None}
    if over:
        cfg = dataclasses.replace(cfg, **over)
    wl = make_workload(cfg, m=m, n=n)
    return wl, oenc.encode(wl.keep, wl.planes, wl.alpha, wl.M, wl.n, exhaustive=exhaustive)


def rel_fro(a, b) -> float:
    a = np.asarray(a, dtype=np.float64)
    b = np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))
