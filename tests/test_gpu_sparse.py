"""Coefficient gradient of sparse cells: two samples per matrix instruction."""
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import TOL_F32
from streamed_shapes import NOT_SPARSE, SPARSE

pytestmark = pytest.mark.gpu


# (test_routes_host.py: which of these are sparse)
@pytest.mark.parametrize("B,n_in,n_out,G", SPARSE + NOT_SPARSE)
def test_coefficient_gradient_of_sparse_cells(oracle, B, n_in, n_out, G):
    g = torch.Generator(device="cpu").manual_seed(91)
    x, gy = torch.randn((B, n_in), generator=g), torch.randn((B, n_out), generator=g)
    want = torch.from_numpy(oracle.backward_coef(x.numpy(), gy.numpy(), G).reshape(G + 1, G + 1, n_in // 2, n_out))
    base = torch.randn(want.shape, generator=g)
    got, added = torch.full(want.shape, float("nan"), device="cuda:0"), base.to("cuda:0")
    for out, flags in ((got, 0), (added, pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF)):
        pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G, flags=flags), x.to("cuda:0"), None, gy.to("cuda:0"), need_grad_x=False, grad_coef=out)
    room = TOL_F32 * want.abs().max().item()
    assert (got.double().cpu() - want).abs().max().item() <= room
    # (the sum is rounded as it meets the base, once, or by the few runs that share a node)
    assert (added.double().cpu() - base.double() - want).abs().max().item() <= room + 2.0 ** -21 * base.abs().max().item()
