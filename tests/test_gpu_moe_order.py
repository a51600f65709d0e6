"""A routed layer's projections of the same rows are the same bits whatever the
form of the large tiles (128 x 128, 128-row halves, whole 256 x 256 tiles) where the
plan does not cut K, and the q/k norm sums a head's squares in one order.  (Another
order would, on a near tie of the router, choose other experts.)  Not so: up to 128
tokens (weight streams, skinny tiles), and where a nearly empty last round is cut
in K; test_plan.py holds the plan to the forms and to the uncut K of these sizes.
"""
import pytest

from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import DeviceLayer, device_batch, to_device_bf16
from synth import LayerConfig, make_weights, make_x
from test_gpu_layer import B, ws_view

pytestmark = pytest.mark.gpu

ROWS = 200  # the smallest batch: 72 rows in its last tile
SIZES = (ROWS, 900, 2100)
# (n, k) of the layer's projections (q/k/v with 4 heads of 128 or 8 of 64; O)
PROJECTIONS = ((4096 + 2 * 512, 2048), (2048, 4096))


@pytest.mark.parametrize("d,hkv,norm,bias", [(128, 4, True, False), (128, 4, False, True),
                                             (64, 8, True, True)])
def test_projections_do_not_depend_on_the_tile_form(d, hkv, norm, bias):
    import torch
    cfg = LayerConfig(hidden=2048, n_q_heads=4096 // d, n_kv_heads=hkv, head_dim=d, n_experts=4,
                      top_k=2, expert_ffn_dim=64, qk_norm=norm, qkv_bias=bias)
    dl = DeviceLayer(cfg, make_weights(cfg, 61))
    x = to_device_bf16(make_x(cfg, 2100, 61))
    got = []
    for n in SIZES:
        k = torch.zeros(1, hkv, 2112, d, dtype=torch.bfloat16, device="cuda")
        v = torch.zeros_like(k)
        db = device_batch(B([0], [0], [n]))
        _, ws = T.layer_prefill(dl.cfg, dl.w, (k, v), db, x[:n].contiguous())
        torch.cuda.synchronize()
        m = T.workspace_layout(dl.cfg, db)
        got.append(dict(k=k[:, :, :ROWS].clone(), v=v[:, :, :ROWS].clone(),
                        q=ws_view(ws, m.q, (ROWS, 4096)).clone(),
                        attn=ws_view(ws, m.attn, (ROWS, 4096)).clone(),
                        x1=ws_view(ws, m.x1, (ROWS, 2048)).clone()))
    assert all(t.abs().amax(-1).min() > 0 for t in got[0].values())
    for other in got[1:]:
        for name, t in other.items():
            assert torch.equal(t, got[0][name]), name
