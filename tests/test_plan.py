"""The launch arithmetic of csrc/plan.hpp, compiled for the host (no GPU, no HIP)."""
import ctypes
import os
import shutil
import subprocess

import pytest

import test_gpu_moe_order as order
from test_gpu_gemm_tiles import CASES

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2606_29629_amd", "csrc")
WRAP = """
#include "plan.hpp"
extern "C" int resid_range(int M, int ld, int row0, int col0, int rows) {
  return tri::resid_range_bytes(M, ld, row0, col0, rows);
}
extern "C" int jobs_of_launch(const int64_t* threads, int first, int n) {
  return tri::jobs_of_launch(threads, first, n);
}
extern "C" int stream_rows(int N, int K, int paired) { return tri::stream_rows(N, K, paired != 0); }
extern "C" void gemm_plan(int M, int N, int K, int swiglu, int tail, int routed, int* out) {
  const tri::GemmPlan p = tri::gemm_plan(M, N, K, swiglu != 0, tail != 0, routed != 0, 256);
  out[0] = p.bm, out[1] = p.bn, out[2] = p.split;
}
extern "C" int moe_tile_rows(int pairs, int experts, int hidden, int ffn) {
  return tri::moe_tile_rows(pairs, experts, hidden, ffn, 256);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "wrap.cpp").write_text(WRAP)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC,
                    str(d / "wrap.cpp"), "-o", str(d / "wrap.so")], check=True)
    return ctypes.CDLL(str(d / "wrap.so"))


@pytest.mark.parametrize("N", [64, 256, 896, 3584, 4100])
@pytest.mark.parametrize("M", [1, 255, 256, 257, 1061, 16384])
def test_residual_prefetch_stays_inside_the_residual(plan, M, N):
    """A 256 x 256 tile's descriptor covers the tile's valid elements and ends
    no later than the tensor (N not a multiple of 256: the last column tile)."""
    for row0 in {0, (M - 1) // 256 * 256}:
        for col0 in range(0, N, 256):
            end = plan.resid_range(M, N, row0, col0, 256)
            rows, cols = min(256, M - row0), min(256, N - col0)
            assert end >= ((rows - 1) * N + cols) * 2
            assert (row0 * N + col0) * 2 + end <= M * N * 2


@pytest.mark.parametrize("threads", [
    [1, 2, 3, 4],
    [2 ** 20, 2 ** 20, 2 ** 30, 2 ** 29],          # one launch
    [2 ** 22, 2 ** 22, 3 * 2 ** 30, 3 * 2 ** 29],  # 256 experts of 3072 x 8192: two
    [2 ** 31, 2 ** 31, 2 ** 31, 2 ** 31],          # each fits, no two do
    [2 ** 32 - 256, 1, 1, 1], [1, 1, 1, 2 ** 32 - 256], [2 ** 33, 1, 1, 1],
])
def test_jobs_of_a_launch_stay_under_the_grid_limit(plan, threads):
    """Every job is launched once, none together with others past 2^32 threads
    (what a launch per job takes is taken together as well)."""
    arr = (ctypes.c_int64 * 4)(*threads)
    first, launches = 0, 0
    while first < 4:
        end = plan.jobs_of_launch(arr, first, 4)
        assert first < end <= 4
        blocks = -(-sum(threads[first:end]) // 256)
        assert end == first + 1 or blocks * 256 < 2 ** 32
        first, launches = end, launches + 1
    assert launches == 1 or sum(threads) > 2 ** 32 - 256


@pytest.mark.parametrize("rows,N,K,paired,stream", [
    # narrow with a long K: the streams took 1.1 to 1.8 times the skinny tiles' time
    (5, 1024, 16384, False, False), (16, 256, 16384, False, False), (16, 1024, 8192, False, False),
    (16, 2048, 8192, False, False), (16, 3584, 18944, False, False), (8, 1024, 8192, True, False),
    (9, 1024, 6144, True, False), (1, 1024, 8192, True, False), (12, 1024, 6144, False, False),
    # the rest: down to 0.7 of it
    (12, 3584, 18944, False, True), (16, 3584, 3584, False, True), (16, 896, 4864, False, True),
    (16, 2048, 4096, False, True), (2, 1024, 8192, False, True), (16, 8192, 8192, False, True),
    (16, 37888, 3584, True, True), (16, 4608, 3584, True, True), (16, 1152, 896, True, True),
    (16, 5120, 2048, True, True), (16, 768, 4096, True, True), (16, 4, 64, False, True),
])
def test_streams_where_they_measured_faster(plan, rows, N, K, paired, stream):
    assert (rows <= plan.stream_rows(N, K, paired)) == stream
    assert 0 <= plan.stream_rows(N, K, paired) <= 16


def gemm_plan(plan, M, N, K, swiglu=False, tail=True, routed=False):
    """(rows, columns, split) of the plan on 256 CUs."""
    out = (ctypes.c_int * 3)()
    plan.gemm_plan(M, N, K, swiglu, tail, routed, out)
    return tuple(out)


@pytest.mark.parametrize("M,N,K", CASES)
def test_gemm_edge_cases_reach_the_forms_they_name(plan, M, N, K):
    assert gemm_plan(plan, M, N, K) == CASES[M, N, K]


def test_routed_sizes_compared_bit_by_bit_differ_in_form_and_keep_k_whole(plan):
    for n, k in order.PROJECTIONS:
        forms = [gemm_plan(plan, m, n, k, routed=True) for m in order.SIZES]
        assert all(split <= 1 for _, _, split in forms)
        assert len(set(forms)) > 1
    # (and the cut that is there: 32 of 288 tiles in the last round)
    assert gemm_plan(plan, 2817, 6144, 2048, routed=True) == (256, 256, 8)


def test_k_parts_fit_the_partials(plan):
    """A K-split's tiles times its parts never exceed the reserved round of 256
    tiles, and no part is empty."""
    for M in (129, 300, 544, 1061, 2817, 4115, 16384):
        for N in (64, 516, 2048, 3584, 9216):
            for K in (64, 448, 4096, 16384, 18944):
                for routed in (False, True):
                    bm, bn, split = gemm_plan(plan, M, N, K, routed=routed)
                    if split > 1:
                        tiles = -(-M // bm) * -(-N // bn)
                        tail = tiles % 256 if tiles > 256 else tiles
                        assert tail * split <= 256
                        assert (split - 1) * -(-(K // 64) // split) < K // 64


@pytest.mark.parametrize("mean,experts,hidden,ffn,rows", [
    (0.25, 128, 2048, 768, 32), (20, 128, 2048, 768, 32), (21, 128, 2048, 768, 128),
    (48, 64, 2048, 1536, 128), (99, 128, 2048, 768, 128), (100, 128, 2048, 768, 256),
    (223, 64, 2048, 1536, 256), (256, 128, 2048, 768, 256),
    (24, 32, 2048, 1024, 32), (25, 32, 2048, 1024, 128),
    (160, 8, 4096, 2048, 128), (212, 8, 4096, 2048, 128), (224, 8, 4096, 2048, 256),
    (160, 8, 4096, 3584, 256), (128, 16, 4096, 1536, 256), (250, 8, 256, 128, 256),
])
def test_expert_tile_rows_where_they_measured_faster(plan, mean, experts, hidden, ffn, rows):
    assert plan.moe_tile_rows(int(mean * experts), experts, hidden, ffn) == rows


def test_expert_tile_rows_of_the_largest_sizes(plan):
    assert plan.moe_tile_rows(2 ** 31 - 1, 256, 8192, 2 ** 20) == 256
    assert plan.moe_tile_rows(2 ** 31 - 1, 1, 64, 64) == 256
    assert plan.moe_tile_rows(1, 1, 64, 64) == 32
