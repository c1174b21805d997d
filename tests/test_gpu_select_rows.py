"""The selection's mask-row scan (grids of more than 64 rows, or masks finer
than the grid) against the oracle, bit for bit: rows whose bytes start and end
off 16-byte boundaries, pixel rows shorter than a 16-byte load, grids of one to
four bit words per row and past them, objects in mask, box and empty mode in
one union, and cell counts that leave the last wave short."""
from dataclasses import replace

import numpy as np
import pytest

from test_gpu_edge import SMALL, _check_select, _session
from harness import OraclePipeline
from workloads import make_weights, to_storage

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m,n,s,n_obj,union", [
    (30, 54, 16, 3, True),      # one word per row, whole 16-byte rows
    (13, 7, 3, 2, True),        # pixel rows of 21 bytes: every start unaligned
    (9, 3, 1, 1, True),         # small grid at stride 1 (the one-wave prior)
    (65, 1, 1, 2, False),       # one column, a row past the one-wave prior
    (5, 130, 5, 3, False),      # three words per row
    (128, 128, 1, 2, True),     # sixteen cells per thread
    (70, 250, 2, 2, True),      # four words, 17,500 cells
    (20, 300, 2, 3, True),      # rows past the bit words (byte map)
    (1100, 2, 2, 1, True),      # more rows than threads
])
def test_mask_rows(m, n, s, n_obj, union):
    cfg = replace(SMALL, m=m, n=n, s=s, n_obj=n_obj, union_objects=union, cap_frames=1, f_max=2, r_s=2)
    W = make_weights(cfg)
    sess, orc = _session(cfg, W), OraclePipeline(cfg, W)
    rng = np.random.default_rng(m * n + s)
    groups = 1 if union else n_obj
    for frame in range(4):
        X = to_storage(rng.standard_normal((1, cfg.mn, cfg.C)).astype(np.float32), "bf16")
        masks = (rng.random((n_obj, m * s, n * s)) < 0.5 / (s * max(m, n))).astype(np.uint8)
        masks[0, -1, -1] = masks[0, 0, 0] = 255     # first and last byte of the mask
        if frame:
            masks[frame % n_obj] = 0                # the cached box, or nothing seen yet
        k = [int(rng.integers(1, max(2, cfg.mn // 3))) for _ in range(groups)]
        _check_select(sess, orc, masks, X, k)
