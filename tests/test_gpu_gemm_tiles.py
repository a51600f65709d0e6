"""The GEMM tile forms at their edges, through tri_linear, against the oracle's
projection in float64 (each element the bf16 rounding of the exact product or
an adjacent value, at most 1% adjacent; see test_gpu_linear.py).

256 x 256 ping-pong tiles: one, two and an odd number of k-tiles; a last M-tile
of 1, 17, 65, 129, 193 rows (every count of active row blocks, of one wave
group or both); a last N-tile of 4 columns (rows not 16-byte aligned: the
narrow stores).  Mid-size 128-row tiles with such rows too.
"""
import numpy as np
import pytest

import oracle
from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import to_device_bf16, to_host_f64
from synth import bf16_to_f32, normal_bf16
from test_gpu_layer import assert_rounded

pytestmark = pytest.mark.gpu

PING = [
    (4097, 4100, 64),    # one k-tile, 1 row and 4 columns in the last tiles
    (4113, 4096, 128),   # two k-tiles, 17 rows
    (4161, 4092, 192),   # three k-tiles, 65 rows, 252 columns
    (4225, 4096, 320),   # 129 rows
    (4289, 3844, 448),   # 193 rows, 4 columns
]
MID = [
    (1061, 768, 9472),   # 256 x 256 tiles split in K, 37 valid rows in the last (partials of those only)
    (300, 516, 4096),    # 128 x 128 tiles split in K, 44 valid rows and 4 columns in the last
    (900, 1280, 2048),   # 128 x 128 tiles, 4 valid rows in the last
    (1400, 4352, 512),   # 128 x 256 tiles
    (200, 700, 256),     # 128 x 128 tiles, rows of 1400 bytes
    (1500, 4076, 256),   # 128 x 256 tiles, rows of 8152 bytes
]


@pytest.mark.parametrize("M,N,K", PING + MID)
def test_gemm_tile_edges(M, N, K):
    import torch
    a_bits, b_bits = normal_bf16(21, 1, (M, K)), normal_bf16(21, 2, (N, K), std=0.05)
    c = T.linear(to_device_bf16(a_bits), to_device_bf16(b_bits))
    torch.cuda.synchronize()
    rows = np.unique(np.r_[np.arange(0, M, 61), np.arange(max(0, M - 260), M)])
    exact = oracle.project(bf16_to_f32(a_bits).astype(np.float64)[rows],
                           bf16_to_f32(b_bits).astype(np.float64))
    assert_rounded(to_host_f64(c)[rows], exact, f"linear {M}x{N}x{K}")
