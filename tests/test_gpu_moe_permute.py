"""The routed order of a step (workspace `perm`): pairs grouped by expert,
ascending within one, at the limits of the one-workgroup permutation (1024
pairs) and of the expert count; the layer's routes for expert counts that are no
multiple of four; and the top-k of logits with ties, -inf and NaN.
"""
import numpy as np
import pytest

from oracle import layer as OL
from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import (DeviceLayer, device_batch, device_cache, to_device_bf16,
                                           to_host_f64)
from synth import LayerConfig, bf16_to_f32, make_cache, make_weights, make_x
from test_gpu_layer import B, ws_view
from test_gpu_moe import routes_agree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,n", [(3, 1, 5), (1, 1, 64), (256, 16, 64), (128, 8, 128), (128, 8, 129),
                                   (65, 4, 1)])
def test_permutation_groups_pairs_by_expert(E, k, n):
    import torch
    cfg = LayerConfig(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, n_experts=E, top_k=k,
                      expert_ffn_dim=64)
    wb = make_weights(cfg, 51)
    if E > 64:
        wb["w_router"][E - 1] = wb["w_router"][0]  # a tie in every token
    kb, vb = make_cache(cfg, n, 64, 51)
    dl = DeviceLayer(cfg, wb)
    db = device_batch(B(list(range(n)), [i % 50 for i in range(n)], [1] * n))
    idx = torch.empty(n, k, dtype=torch.int32, device="cuda")
    w = torch.empty(n, k, dtype=torch.float32, device="cuda")
    _, ws = T.layer_decode(dl.cfg, dl.w, device_cache(kb, vb), db,
                           to_device_bf16(make_x(cfg, n, 51)), route_idx=idx, route_w=w)
    torch.cuda.synchronize()
    m = T.workspace_layout(dl.cfg, db)
    perm = ws[m.perm:m.perm + 4 * n * k].view(torch.int32).cpu().numpy()
    idx, w = idx.cpu().numpy(), w.cpu().numpy()
    assert np.array_equal(perm, np.argsort(idx.ravel(), kind="stable"))
    assert idx.min() >= 0 and idx.max() < E
    assert all(len(set(row)) == k for row in idx.tolist())
    assert np.all(np.diff(w, axis=1) <= 0) and np.allclose(w.sum(1), 1, atol=1e-5)
    if E > 64:  # the duplicated expert: never ahead of its lower twin
        for row in idx.tolist():
            assert E - 1 not in row or (0 in row and row.index(0) < row.index(E - 1))


@pytest.mark.parametrize("E,k,finite", [(8, 5, 2), (70, 16, 4), (256, 3, 1), (8, 8, 0)])
def test_topk_of_infinite_logits(E, k, finite):
    """Distinct experts, in descending order with ties to the lower index, also
    where fewer than k logits are above -inf; NaN logits come last."""
    import torch
    cfg = LayerConfig(hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, n_experts=E, top_k=k,
                      expert_ffn_dim=64)
    h = torch.zeros(3, 256, device="cuda")
    h[:, 0] = 1.0  # the logits are the router's first column
    col = torch.full((E,), -float("inf"))
    chosen = [(5 * i + 3) % E for i in range(finite)]
    col[chosen] = torch.arange(finite, 0, -1).float()
    for nan in (False, True):
        wr = torch.zeros(E, 256, dtype=torch.bfloat16, device="cuda")
        if nan:
            col[E - 1] = float("nan")
        wr[:, 0] = col.to(torch.bfloat16).cuda()
        idx = torch.empty(3, k, dtype=torch.int32, device="cuda")
        w = torch.empty(3, k, dtype=torch.float32, device="cuda")
        T.moe_route(T.make_config(cfg), h, wr, idx, w)
        torch.cuda.synchronize()
        rest = [e for e in range(E) if e not in chosen and not (nan and e == E - 1)]
        want = (chosen + rest + [E - 1] * nan)[:k]
        assert idx.tolist() == [want] * 3
        if finite and not nan:
            assert torch.all(w[:, finite:] == 0) and torch.allclose(w.sum(1).cpu(), torch.ones(3))


@pytest.mark.parametrize("E,k,hidden,n", [(17, 4, 1024, 9), (3, 3, 1024, 70), (65, 4, 512, 40),
                                          (1, 1, 256, 5), (255, 16, 448, 200), (18, 2, 320, 129)])
def test_layer_routes_of_any_expert_count(E, k, hidden, n):
    """The router's logits as the layer forms them (from its own bf16 h2): the
    routes and weights of every token against float64."""
    import torch
    cfg = LayerConfig(hidden=hidden, n_q_heads=2, n_kv_heads=1, head_dim=64, n_experts=E, top_k=k,
                      expert_ffn_dim=64)
    wb = make_weights(cfg, 52)
    kb, vb = make_cache(cfg, n, 64, 52)
    dl = DeviceLayer(cfg, wb)
    db = device_batch(B(list(range(n)), [i % 50 for i in range(n)], [1] * n))
    idx = torch.empty(n, k, dtype=torch.int32, device="cuda")
    w = torch.empty(n, k, dtype=torch.float32, device="cuda")
    need = T.workspace_size(dl.cfg, db)
    buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    T.layer_decode(dl.cfg, dl.w, device_cache(kb, vb), db, to_device_bf16(make_x(cfg, n, 52)),
                   workspace=buf[:need], route_idx=idx, route_w=w)
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0xA5).all())
    m = T.workspace_layout(dl.cfg, db)
    h2 = to_host_f64(ws_view(buf, m.h2, (n, hidden)))
    logits = h2 @ bf16_to_f32(wb["w_router"]).astype(np.float64).T
    got = idx.cpu().numpy().astype(np.int64)
    routes_agree(got, logits, k, 1e-5)  # (fp32 sums: near ties may swap)
    p = OL.softmax(np.take_along_axis(logits, got, 1))  # renormalised over the chosen
    assert np.allclose(w.cpu().numpy(), p, rtol=1e-4, atol=1e-6)
