"""The GEMM tile forms at their edges, through tri_linear, against the oracle's
projection in float64 (each element the bf16 rounding of the exact product or
an adjacent value, at most 1% adjacent; see test_gpu_linear.py).

Each case says which form it reaches (rows, columns, split: 1 whole tiles, 0 the
last round as 128-row halves, more K-parts of the last round); test_plan.py
holds the plan to it.
"""
import numpy as np
import pytest

import oracle
from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import to_device_bf16, to_host_f64
from synth import bf16_to_f32, normal_bf16
from test_gpu_layer import assert_rounded

pytestmark = pytest.mark.gpu

CASES = {
    # 256 x 256 tiles, the staggered loop: one, two, three, odd numbers of k-tiles; a
    # last M-tile of 1, 17, 65, 129, 145, 193 and all rows (every count of active row
    # blocks, of one wave group or both); a last N-tile of 4 columns (rows not 16-byte
    # aligned: the narrow stores) and of 252
    (4097, 4100, 64): (256, 256, 1),
    (4113, 4096, 128): (256, 256, 1),
    (4161, 4092, 192): (256, 256, 1),
    (3841, 3844, 64): (256, 256, 1),
    (3969, 4096, 320): (256, 256, 1),
    (3985, 3844, 192): (256, 256, 1),
    (4033, 3844, 448): (256, 256, 1),
    (4096, 4096, 128): (256, 256, 1),
    # the last round of them as 128-row halves, one of 1 row, one of 65
    (4225, 4096, 320): (256, 256, 0),
    (4289, 3844, 448): (256, 256, 0),
    (1400, 4352, 512): (256, 256, 0),
    (1500, 4076, 256): (256, 256, 0),   # rows of 8152 bytes
    # the last round in K-parts, after whole rounds (15 valid rows and 52 columns in
    # the last tile) and alone (19 rows, 244 columns)
    (5903, 2612, 1728): (256, 256, 7),
    (4115, 500, 6016): (256, 256, 5),
    # 128 x 256 tiles: 7 and 28 valid rows in the last
    (3079, 2360, 320): (128, 256, 1),
    (3100, 2372, 320): (128, 256, 1),
    # 128 x 128 tiles in K-parts: 37 valid rows; 44 valid rows and 4 columns
    (1061, 768, 9472): (128, 128, 4),
    (300, 516, 4096): (128, 128, 8),
    # 128 x 128 tiles: 4 valid rows; rows of 1400 bytes
    (900, 1280, 2048): (128, 128, 1),
    (200, 700, 256): (128, 128, 1),
}


@pytest.mark.parametrize("M,N,K", CASES)
def test_gemm_tile_edges(M, N, K):
    import torch
    a_bits, b_bits = normal_bf16(21, 1, (M, K)), normal_bf16(21, 2, (N, K), std=0.05)
    c = T.linear(to_device_bf16(a_bits), to_device_bf16(b_bits))
    torch.cuda.synchronize()
    rows = np.unique(np.r_[np.arange(0, M, 61), np.arange(max(0, M - 260), M)])
    exact = oracle.project(bf16_to_f32(a_bits).astype(np.float64)[rows],
                           bf16_to_f32(b_bits).astype(np.float64))
    assert_rounded(to_host_f64(c)[rows], exact, f"linear {M}x{N}x{K}")
