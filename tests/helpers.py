"""Shared helpers of the GPU parity tests: workload definitions and comparison metrics."""
from __future__ import annotations

import numpy as np
import torch

from oracle import rtn_oracle as O
from paper_2505_15909_amd import synth

REL_FRO_TOL = 2e-3       # relative Frobenius error bound of the linear layer
MAX_ABS_TOL = 1e-2       # max abs error bound, taken literally ...
HALF_ULP_REL = 2.0 ** -11  # ... except in the cases listed below, which get one fp16 rounding of the result on top

# The only cases where the literal max-abs bound cannot hold: outputs so large that the fp16 output format itself uses
# up the bound.  For |C| in [16, 32) the half-ulp is 7.8e-3, which leaves 2.2e-3 for everything else (measured: up to
# 1.08e-2 in total at |C| = 30 on the path that rounds each dequantised weight to fp16 first); from |C| = 32 the half-ulp
# is 1.6e-2 and a correctly rounded result already misses 1e-2.  Keyed by the `allow` tag the test passes; each entry
# states where such outputs come from.  Everything else, and the listed cases while |C| stays below 16, is held to
# max|dC| <= 1e-2.
FP16_OUTPUT_ALLOWANCE = {
    "llama70b_down": "70B-shaped down projection, K = 28672, heavy-tailed weights with 1 % of input columns x10: "
                     "|C| reaches 23-35 depending on the batch",
}


def linear_errors(C_gpu: np.ndarray, C_ref: np.ndarray):
    d = C_gpu.astype(np.float64) - C_ref
    fro = float(np.linalg.norm(d) / max(np.linalg.norm(C_ref), 1e-300))
    max_abs = float(np.max(np.abs(d))) if d.size else 0.0
    excess = float(np.max(np.abs(d) - (MAX_ABS_TOL + HALF_ULP_REL * np.abs(C_ref)))) if d.size else -1.0
    return fro, max_abs, excess


def assert_linear_close(C_gpu, C_ref, what="", allow=None):
    """rel Frobenius <= 2e-3 and max abs <= 1e-2 (literal).  allow: a key of FP16_OUTPUT_ALLOWANCE for the listed cases
    whose outputs reach 16 and more in magnitude; where they do, the case is held to 1e-2 + 2^-11 |C_ref| instead."""
    fro, max_abs, excess = linear_errors(C_gpu, C_ref)
    assert fro <= REL_FRO_TOL, f"{what}: rel Frobenius {fro:.3e} > {REL_FRO_TOL}"
    c_max = float(np.max(np.abs(C_ref))) if C_ref.size else 0.0
    if allow is not None:
        assert allow in FP16_OUTPUT_ALLOWANCE, allow
    if allow is None or c_max < 16.0:      # a listed case still gets the literal bound while its outputs stay below 16
        assert max_abs <= MAX_ABS_TOL, f"{what}: max abs {max_abs:.3e} > 1e-2 (|C_ref| up to {c_max:.2f})"
    else:
        assert excess <= 0.0, f"{what}: max abs {max_abs:.3e} exceeds 1e-2 + 2^-11 |C| (|C_ref| up to {c_max:.2f})"
    return fro, max_abs


def tile_rows(row_tiles, N):
    """Row indices of the given 16-row tiles."""
    rows = np.concatenate([np.arange(t * 16, t * 16 + 16) for t in row_tiles])
    assert rows.max() < N
    return rows


def packed_rows_image(packed: np.ndarray, row_tiles, K: int, bits: int) -> np.ndarray:
    """Bytes of the given row tiles from a full packed image (tiles are row-tile-major)."""
    per_tile_row = 16 * K * bits // 8
    return np.concatenate([packed[t * per_tile_row:(t + 1) * per_tile_row] for t in row_tiles])


def pick_row_tiles(N: int, count: int, seed: int):
    NT = N // 16
    if NT <= count:
        return np.arange(NT)
    rng = np.random.default_rng(seed)
    picks = set(rng.choice(NT, size=count - 2, replace=False).tolist())
    picks.update([0, NT - 1])                                   # always the first and last tile row
    return np.array(sorted(picks))


def make_weight(cfg_dist: str, N: int, K: int, seed: int, device):
    if cfg_dist == "normal02":
        return synth.normal_weight(N, K, 0.02, seed, device)
    if cfg_dist == "normal01":
        return synth.normal_weight(N, K, 0.01, seed, device)
    if cfg_dist == "heavy":
        return synth.heavy_tail_weight(N, K, 0.02, seed, device)
    raise ValueError(cfg_dist)


# Layers (N, K of each module) for the launches that rtn_layer_forward merges: what test_host_plans.py asserts of their plans is
# what the GPU tests on the same lists rely on.
LAYER_RAGGED = [(48, 1024), (272, 4096), (16, 1024), (2064, 2048), (80, 14336)]
LAYER_2048 = [(3072, 2048), (2048, 2048), (16384, 2048), (2048, 8192)]

# (M, N, K, bits, g) with zero points that the wide kernel runs: row blocks of 32, 48 and 64 rows, all group sizes, with and without a K split.
WIDE_ZERO_POINTS = [(17, 304, 512, 4, 0), (21, 304, 1536, 4, 128), (40, 304, 1536, 4, 256), (33, 304, 512, 4, 128), (130, 2576, 1536, 4, 32),
                    (491, 528, 512, 4, 32), (130, 2576, 1024, 4, 64), (491, 528, 512, 4, 64), (100, 304, 1536, 4, 128), (60, 304, 512, 4, 0),
                    (17, 304, 256, 8, 0), (130, 528, 2048, 8, 0), (200, 528, 2048, 8, 0), (21, 16400, 256, 8, 32), (33, 16400, 256, 8, 64),
                    (491, 1040, 256, 8, 32), (200, 2576, 256, 8, 64), (21, 304, 256, 8, 128), (130, 1040, 2048, 8, 128), (60, 304, 256, 8, 128)]

# Layers whose modules (M, N, K, bits, g) share launches of the block (3) or tile kernel (4) with a workspace of 256 MiB, and how many of
# them have K split in a shared launch: two splits and more put partial sums behind one another in the workspace.
SHARED_LAYERS = [(3, 2, [(100, 272, 14336, 4, 128), (101, 288, 14336, 4, 128)]),
                 (3, 2, [(20, 272, 14336, 8, 0), (21, 288, 14336, 8, 0)]),
                 (3, 3, [(40, 272, 14336, 4, 32), (41, 288, 14336, 4, 32), (42, 304, 14336, 4, 32)]),
                 (3, 2, [(200, 272, 14336, 4, 64), (201, 288, 14336, 4, 64)]),
                 (3, 2, [(100, 272, 8192, 8, 64), (101, 288, 8192, 8, 64)]),
                 (3, 0, [(33 + i, 272 + 16 * i, 4096, 4, 32) for i in range(11)]),          # eight and three
                 (4, 2, [(1040, 2064, 14336, 4, 128), (1041, 2080, 14336, 4, 0)]),
                 (4, 2, [(1100 + i, 4112 + 16 * i, 4096, 8, 128) for i in range(4)])]

# Launches of the block kernel with row tiles of two heights, which have more than 256 workgroups: explicit configurations (M, N, K, bits, g):
# (m_rows16, wavefronts along K, K splits); automatic plans with zero points; and layers whose modules share the launch.
TWO_HEIGHTS = {(129, 33040, 512, 4, 128): (8, 1, 1), (200, 33040, 512, 4, 128): (8, 1, 1), (200, 33040, 512, 8, 0): (8, 1, 1),
               (200, 16528, 1024, 8, 128): (8, 2, 1), (129, 16528, 1536, 4, 256): (8, 2, 1), (300, 8272, 2048, 4, 128): (8, 4, 1), (300, 11296, 1536, 4, 0): (8, 1, 2),
               (270, 13328, 1024, 4, 32): (4, 1, 1), (270, 6672, 1024, 8, 64): (4, 2, 1), (270, 3344, 2048, 4, 64): (4, 4, 1),
               (80, 4176, 4096, 4, 128): (4, 8, 1), (80, 4176, 2304, 8, 32): (4, 8, 1)}
TWO_HEIGHTS_ZP = [(129, 33040, 512, 4, 128), (129, 33040, 512, 4, 32), (200, 33040, 512, 8, 128), (200, 33040, 512, 4, 128), (300, 41232, 512, 4, 64)]
TWO_HEIGHTS_LAYERS = [[(M + i, N, K, bits, g) for i, (N, K) in enumerate([(4112, 1024), (8208, 1024), (16400, 1024), (4112, 2048)])]
                      for M, bits, g in ((129, 4, 128), (200, 4, 64), (300, 4, 128), (300, 8, 128))]

# Grouped calls of modules of up to 16 rows that share a launch of the block kernel instead of the small-batch kernel's, and the modules
# that do: (members, [(M, N, K, bits, g)]).
GROUPED_ON_BLOCKS = [([0, 1, 2, 3], [(16, 528, 7168, 4, 64), (9, 528, 7168, 4, 64), (12, 512, 7168, 4, 64), (16, 544, 7168, 4, 64)]),
                     ([0, 2, 3], [(16, 528, 14336, 8, 0), (1, 512, 14336, 8, 0), (9, 544, 14336, 8, 0), (12, 528, 14336, 8, 0)]),
                     ([], [(4, 1024, 2048, 4, 128)] * 4)]

# Alike modules of a grouped call that go to the block kernel in two launches: (N, K, bits, g), rows, modules of the first launch.
GROUPED_IN_TWO_LAUNCHES = [((400, 7168, 4, 0), [11, 9, 11, 15, 14, 8, 14, 16, 3, 12, 3, 12, 12, 2, 14, 15], 8),
                           ((592, 6144, 8, 0), [11, 14, 7, 13, 5, 13, 2, 14, 14, 11, 5, 7, 15, 4, 10], 7),
                           ((2416, 13824, 4, 128), [4, 16, 5, 9, 12, 7, 16, 3, 14, 10, 11], 5)]

# (M, N, K, bits, g) with zero points that the block kernel runs, and its 32-row blocks and wavefronts along K.
BLOCK_ZERO_POINTS = {(70, 1040, 4096, 4, 128): (1, 1), (33, 304, 1024, 4, 0): (1, 2), (20, 304, 2048, 4, 128): (1, 4), (250, 8208, 1024, 4, 32): (2, 1),
                     (128, 304, 1024, 4, 128): (2, 2), (250, 304, 2048, 4, 128): (2, 4), (161, 12304, 1024, 4, 32): (3, 2),
                     (90, 12304, 2048, 4, 32): (3, 4), (230, 16400, 1024, 4, 32): (4, 1), (230, 8208, 4096, 4, 128): (4, 2),
                     (70, 304, 2048, 8, 128): (1, 1), (20, 304, 1024, 8, 0): (1, 4), (100, 304, 2048, 8, 0): (2, 1), (250, 4112, 1024, 8, 64): (2, 2),
                     (100, 304, 1024, 8, 128): (2, 4), (161, 12304, 1024, 8, 64): (3, 2), (90, 8208, 2048, 8, 32): (3, 4),
                     (230, 16400, 1024, 8, 32): (4, 1), (230, 8208, 4096, 8, 0): (4, 2)}
