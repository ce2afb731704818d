"""Coefficient gradients of streams that are cut into runs: nodes that a run owns are written, those it shares
with another are cleared and added to."""
import numpy as np
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import TOL_F32

pytestmark = pytest.mark.gpu

# more rows than a workgroup sorts for itself, one block, few pairs: always a cut stream.  From three million entries of
# the gradient on only the shared nodes are cleared.
SHAPES = [(8193, 2, 64, 3), (8200, 4, 33, 64), (12288, 100, 262, 16), (9000, 44, 132, 33),
          (8193, 40, 128, 35), (12288, 40, 132, 40), (9001, 60, 132, 64)]   # (from G = 40 on: the walk)


def _rows(kind, B, n_in, g):
    x = torch.randn((B, n_in), generator=g)
    if kind == "one cell":
        return x * 0 + 0.1
    if kind == "corners":        # the first and the last cells, nothing between
        return torch.where(x > 0.5, 4.2, -4.2)
    if kind == "clusters":       # runs end inside a cell and next to wide gaps
        return torch.randn(7, generator=g)[torch.randint(7, (B, n_in), generator=g)]
    return x


@pytest.mark.parametrize("B,n_in,n_out,G", SHAPES)
@pytest.mark.parametrize("kind", ["spread", "one cell", "corners", "clusters"])
def test_runs_of_a_stream_write_every_node_once(oracle, B, n_in, n_out, G, kind):
    """Into a gradient of NaN, and added to one; by the stream alone and, beside grad_x, by the walk where the grid
    is fine.  (grad_y is positive: a sum of N terms of one sign, rounded like a random walk of a quarter of
    them each, is good to sqrt(N / 4) 2^-24 < 4e-6 of itself.)"""
    dev = torch.device("cuda:0")
    g = torch.Generator(device="cpu").manual_seed(83)
    x, gy = _rows(kind, B, n_in, g), torch.rand((B, n_out), generator=g) + 0.5
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g)
    want = oracle.backward_coef(x.numpy(), gy.numpy(), G).reshape(P.shape)
    x, gy, P = x.to(dev), gy.to(dev), P.to(dev)
    for grad_x in (False, True):
        got = torch.full(P.shape, float("nan"), device=dev)
        pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G), x, P, gy, need_grad_x=grad_x, grad_coef=got)
        added = P.clone()
        pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G, flags=pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF), x, P, gy,
                           need_grad_x=grad_x, grad_coef=added)
        torch.cuda.synchronize()
        got, added, base = (t.double().cpu().numpy() for t in (got, added, P))
        assert (got[want == 0.0] == 0.0).all() and (added == base)[want == 0.0].all()
        room = TOL_F32 * np.abs(want).max()
        assert np.abs(got - want).max() <= room, (grad_x, np.abs(got - want).max(), np.abs(want).max())
        # (and the sum is rounded as it meets the base: once, or by the few runs that share a node)
        assert np.abs(added - base - want).max() <= room + 2.0 ** -21 * np.abs(base).max(), grad_x
