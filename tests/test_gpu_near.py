"""Forward pass on grids whose slab fits LDS once: workgroups that share lines lie side by side and bring the next slab near."""
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import TOL_F32, rowwise_rel_err

pytestmark = pytest.mark.gpu


# one to five tiles of 16 outputs in a block of four and behind it, one to five tiles of 4096 rows, the last one ragged; runs of many
# pairs and of few; either side of the rule (rows per tile against nodes); both ends of the range of grids
@pytest.mark.parametrize("B,n_in,n_out,G", [(8192, 48, 16, 35), (4100, 90, 33, 36), (1030, 120, 48, 35), (17000, 30, 100, 40),
                                            (9000, 64, 72, 41), (12288, 44, 130, 49), (5000, 100, 256, 44), (1000, 64, 40, 48)])
def test_forward_with_the_next_slab_brought_near(oracle, B, n_in, n_out, G):
    g = torch.Generator(device="cpu").manual_seed(17)
    x, P = torch.randn((B, n_in), generator=g), torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g)
    packed = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G), P.to("cuda:0"))
    y = torch.full((B, n_out), float("nan"), device="cuda:0")
    pkg.lmkan_forward(pkg.LayerDesc(n_in, n_out, G, coef_layout=pkg.LMKAN_LAYOUT_PACKED), x.to("cuda:0"), packed, y=y)
    want = oracle.forward(x.numpy(), P.numpy(), G, threads=8)
    assert rowwise_rel_err(y.cpu().numpy(), want) <= TOL_F32
