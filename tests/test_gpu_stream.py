"""Short-batch projections as weight streams (at most 16 tokens), at the sizes
where they can go wrong: fewer k-tiles than waves, one row, 8 / 9 and 16 / 17
tokens (the limits of the forms), a last block of 4 weight rows, more blocks
than resident workgroups, and the rows at which a narrow matrix with a long K takes
the skinny tiles instead.  tri_linear against the oracle's projection, and
every stage of a layer step (q/k/v, O, gate/up with its own RMSNorm, down) on
identical inputs; tolerances as in test_gpu_layer.py (1 bf16 ulp).
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import to_device_bf16, to_host_f64
from synth import LayerConfig, bf16_to_f32, layer_c1, layer_talker, normal_bf16
from test_gpu_layer import B, Case, assert_rounded, check_down, stage_parity

pytestmark = pytest.mark.gpu

LINEAR = [(1, 4, 64), (3, 36, 128), (8, 516, 448), (9, 260, 576), (16, 1000, 4096),
          (2, 20004, 320), (13, 24580, 192), (2, 516, 8192), (3, 516, 8192), (16, 260, 12288)]


@pytest.mark.parametrize("M,N,K", LINEAR)
def test_stream_linear(M, N, K):
    import torch
    a_bits, b_bits = normal_bf16(31, 1, (M, K)), normal_bf16(31, 2, (N, K), std=0.05)
    c = T.linear(to_device_bf16(a_bits), to_device_bf16(b_bits))
    torch.cuda.synchronize()
    exact = oracle.project(bf16_to_f32(a_bits).astype(np.float64),
                           bf16_to_f32(b_bits).astype(np.float64))
    assert_rounded(to_host_f64(c), exact, f"stream linear {M}x{N}x{K}")


D128 = LayerConfig(hidden=512, n_q_heads=5, n_kv_heads=1, head_dim=128, ffn_dim=1088, qkv_bias=True)
LONG = LayerConfig(hidden=6144, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=64, qk_norm=True)
WIDE = LayerConfig(hidden=4096, n_q_heads=2, n_kv_heads=1, head_dim=64, ffn_dim=192)


@pytest.mark.parametrize("cfg,n", [(layer_c1(), 1), (layer_c1(), 9), (D128, 3), (D128, 8), (D128, 16),
                                   (D128, 17), (WIDE, 4), (WIDE, 5), (LONG, 2), (LONG, 3),
                                   (dataclasses.replace(layer_talker(), qkv_bias=True), 1),
                                   (dataclasses.replace(D128, qk_norm=True), 7)])
def test_stream_layer_stages(cfg, n):
    batch = B(list(range(n))[::-1], [7 * i % 60 for i in range(n)], [1] * n)
    cs = Case(cfg, batch, n, 64, seed=41)
    out, ws = cs.run(decode=True)
    rows = np.arange(n)
    x1, act, w = stage_parity(cs, ws, rows, label=f"stream {cfg.hidden} n={n}")
    check_down(cs, out, x1, act, w, rows, f"stream {cfg.hidden} n={n}")


def test_stream_prefill_of_few_tokens():
    """Two short prompts of one call (their tokens share the projections)."""
    cs = Case(D128, B([1, 0], [0, 11], [5, 2]), 2, 64, seed=42)
    out, ws = cs.run()
    rows = np.arange(7)
    x1, act, w = stage_parity(cs, ws, rows, label="stream prefill")
    check_down(cs, out, x1, act, w, rows, "stream prefill")


@pytest.mark.parametrize("hidden,heads,n", [(192, 3, 1), (192, 3, 16), (960, 15, 16), (64, 1, 17)])
def test_stream_qk_norm_of_odd_hidden_stays_in_its_workspace(hidden, heads, n):
    """K not cut (hidden an odd multiple of 64): the normed q/k/v's fp32 plane,
    in a workspace of exactly its size with a pattern behind it."""
    import torch
    cfg = LayerConfig(hidden=hidden, n_q_heads=heads, n_kv_heads=heads, head_dim=64, ffn_dim=320,
                      qk_norm=True)
    cs = Case(cfg, B(list(range(n)), [3 * i % 20 for i in range(n)], [1] * n), n, 64, seed=43)
    need = T.workspace_size(cs.dl.cfg, cs.db)
    buf = torch.full((need + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
    out, ws = T.layer_decode(cs.dl.cfg, cs.dl.w, cs.cache, cs.db, cs.x, workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xA5).all())
    rows = np.arange(n)
    x1, act, w = stage_parity(cs, ws, rows, label=f"stream qk-norm {hidden} n={n}")
    check_down(cs, out, x1, act, w, rows, f"stream qk-norm {hidden} n={n}")
