"""Workgroups whose tiles of outputs share lines of the table lie side by side, and bring the next slab near where one fits LDS."""
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import TOL_F32, rowwise_rel_err
from streamed_shapes import NEAR, NOT_NEAR, SIDE_BY_SIDE, SIDE_BY_SIDE_BF16

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


# (test_routes_host.py: these reach the kernels that place their tiles of outputs by the lines they share)
@pytest.mark.parametrize("B,n_in,n_out,G,layout,dtype", [(*shape, torch.float32) for shape in SIDE_BY_SIDE] +
                         [(*shape, pkg.LMKAN_LAYOUT_PACKED, torch.bfloat16) for shape in SIDE_BY_SIDE_BF16])
def test_both_directions_with_tiles_that_share_lines_side_by_side(oracle, B, n_in, n_out, G, layout, dtype):
    g = torch.Generator(device="cpu").manual_seed(18)
    x, gy = torch.randn((B, n_in), generator=g), torch.randn((B, n_out), generator=g)
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g).to(dtype)
    code = pkg.LMKAN_F32 if dtype == torch.float32 else pkg.LMKAN_BF16
    table = P.to("cuda:0")
    if layout == pkg.LMKAN_LAYOUT_PACKED:
        table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=code), table)
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=code, coef_layout=layout)
    y = pkg.lmkan_forward(desc, x.to("cuda:0"), table)
    gx, _ = pkg.lmkan_backward(desc, x.to("cuda:0"), table, gy.to("cuda:0"), need_grad_coef=False)
    stored = P.float().numpy()
    assert rowwise_rel_err(y.cpu().numpy(), oracle.forward(x.numpy(), stored, G, threads=8)) <= TOL_F32
    want = oracle.backward_input(x.numpy(), stored, gy.numpy(), G)
    assert rowwise_rel_err(gx.cpu().numpy(), want) <= TOL_F32
