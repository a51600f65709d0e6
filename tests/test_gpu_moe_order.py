"""A routed layer's projections of the same rows are the same bits whatever the
tile form (128 x 128, 128-row halves, whole 256 x 256 tiles): the sum over K is
not cut, and the q/k norm sums a head's squares in one order.  (Another order
would, on a near tie of the router, choose other experts.)
"""
import pytest

from paper_2606_29629_amd import _lib as T
from paper_2606_29629_amd.workload import DeviceLayer, device_batch, to_device_bf16
from synth import LayerConfig, make_weights, make_x
from test_gpu_layer import B

pytestmark = pytest.mark.gpu

ROWS = 200  # the smallest batch: 72 rows in its last tile


@pytest.mark.parametrize("d,hkv,norm,bias", [(128, 4, True, False), (128, 4, False, True),
                                             (64, 8, True, True)])
def test_projections_do_not_depend_on_the_tile_form(d, hkv, norm, bias):
    import torch
    cfg = LayerConfig(hidden=2048, n_q_heads=4096 // d, n_kv_heads=hkv, head_dim=d, n_experts=4,
                      top_k=2, expert_ffn_dim=64, qk_norm=norm, qkv_bias=bias)
    dl = DeviceLayer(cfg, make_weights(cfg, 61))
    x = to_device_bf16(make_x(cfg, 2100, 61))
    got = []
    for n in (ROWS, 900, 2100):
        k = torch.zeros(1, hkv, 2112, d, dtype=torch.bfloat16, device="cuda")
        v = torch.zeros_like(k)
        T.layer_prefill(dl.cfg, dl.w, (k, v), device_batch(B([0], [0], [n])), x[:n].contiguous())
        torch.cuda.synchronize()
        got.append((k[:, :, :ROWS].clone(), v[:, :, :ROWS].clone()))
    assert got[0][0].abs().amax(-1).min() > 0 and got[0][1].abs().amax(-1).min() > 0
    for k, v in got[1:]:
        assert torch.equal(k, got[0][0]) and torch.equal(v, got[0][1])
