"""Workgroups whose tiles of outputs share lines of the table lie side by side, and bring the next slab near where one fits LDS."""
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import TOL_F32, rowwise_rel_err
from streamed_shapes import NEAR, NOT_NEAR

pytestmark = pytest.mark.gpu


# (test_routes_host.py: which of these bring the next slab near)
@pytest.mark.parametrize("B,n_in,n_out,G", NEAR + NOT_NEAR)
def test_forward_with_the_next_slab_brought_near(oracle, B, n_in, n_out, G):
    g = torch.Generator(device="cpu").manual_seed(17)
    x, P = torch.randn((B, n_in), generator=g), torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g)
    packed = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G), P.to("cuda:0"))
    y = torch.full((B, n_out), float("nan"), device="cuda:0")
    pkg.lmkan_forward(pkg.LayerDesc(n_in, n_out, G, coef_layout=pkg.LMKAN_LAYOUT_PACKED), x.to("cuda:0"), packed, y=y)
    want = oracle.forward(x.numpy(), P.numpy(), G, threads=8)
    assert rowwise_rel_err(y.cpu().numpy(), want) <= TOL_F32


# tiles of 16 outputs (float32) in groups of four and a rest, of 32 (bfloat16 input gradient) in pairs and a rest, pairs split or not
@pytest.mark.parametrize("B,n_in,n_out,G,dtype", [(9000, 60, 33, 25, torch.float32), (2000, 120, 72, 33, torch.float32),
                                                  (1500, 200, 130, 28, torch.float32), (700, 180, 96, 24, torch.bfloat16),
                                                  (2600, 90, 161, 30, torch.bfloat16), (1100, 100, 32, 17, torch.bfloat16)])
def test_both_directions_with_tiles_that_share_lines_side_by_side(oracle, B, n_in, n_out, G, dtype):
    g = torch.Generator(device="cpu").manual_seed(18)
    x, gy = torch.randn((B, n_in), generator=g), torch.randn((B, n_out), generator=g)
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g).to(dtype)
    code = pkg.LMKAN_F32 if dtype == torch.float32 else pkg.LMKAN_BF16
    packed = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=code), P.to("cuda:0"))
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=code, coef_layout=pkg.LMKAN_LAYOUT_PACKED)
    y = pkg.lmkan_forward(desc, x.to("cuda:0"), packed)
    gx, _ = pkg.lmkan_backward(desc, x.to("cuda:0"), packed, gy.to("cuda:0"), need_grad_coef=False)
    stored = P.float().numpy()
    assert rowwise_rel_err(y.cpu().numpy(), oracle.forward(x.numpy(), stored, G, threads=8)) <= TOL_F32
    want = oracle.backward_input(x.numpy(), stored, gy.numpy(), G)
    assert rowwise_rel_err(gx.cpu().numpy(), want) <= TOL_F32
