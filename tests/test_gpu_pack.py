"""lmkan_pack at the shapes where its workgroups take all outputs, a part of them, and a ragged last part."""
import pytest
import torch

import paper_2509_07103_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n_in,n_out,G", [(2, 1, 3), (2, 64, 64), (2, 65536, 16), (2, 8321, 64), (6, 4099, 3), (40, 1000, 5),
                                          (600, 333, 20)])
def test_pack_matches_a_copy(n_in, n_out, G, dtype):
    dev = torch.device("cuda:0")
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=pkg.LMKAN_F32 if dtype == torch.float32 else pkg.LMKAN_BF16)
    P = torch.randn(desc.coef_shape(), device=dev).to(dtype)
    K, tiles, nodes = n_in // 2, (n_out + 63) // 64, (G + 1) ** 2
    want = torch.nn.functional.pad(P.view(nodes, K, n_out), (0, tiles * 64 - n_out)).view(nodes, K, tiles, 64)
    assert torch.equal(pkg.lmkan_pack(desc, P).view(tiles, K, nodes, 64), want.permute(2, 1, 0, 3))
