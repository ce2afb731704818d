"""Input gradient of 16-bit tables on the matrix cores (gy in three parts) against the oracle: edges of its tiles,
magnitudes at the ends of the range, values that are not finite."""
import numpy as np
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import ORACLE_DTYPE, TOL_F32, bits, rowwise_rel_err

pytestmark = pytest.mark.gpu
DTYPE = {"f16": (pkg.LMKAN_F16, torch.float16), "bf16": (pkg.LMKAN_BF16, torch.bfloat16)}


def _layer(B, n_in, n_out, G, storage, layout, seed=5):
    gen = torch.Generator(device="cpu").manual_seed(seed)
    x = torch.randn((B, n_in), generator=gen) * 1.5
    P = (torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=gen) * 0.1).to(DTYPE[storage][1]).cuda()
    gy = torch.randn((B, n_out), generator=gen)
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0])
    if layout == "packed":
        table = pkg.lmkan_pack(desc, P)
        desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0], coef_layout=pkg.LMKAN_LAYOUT_PACKED)
    else:
        table = P
    return x, P, table, gy, desc


def _grad_x(desc, x, table, gy):
    gx, _ = pkg.lmkan_backward(desc, x.cuda(), table, gy.cuda(), need_grad_coef=False)
    torch.cuda.synchronize()
    return gx.cpu().numpy()


@pytest.mark.parametrize("B,n_in,n_out,G,storage,layout", [
    # tiles of 512 rows x 64 outputs (float16, G <= 16; either layout)
    (511, 300, 128, 3, "f16", "packed"), (513, 300, 129, 16, "f16", "packed"), (1537, 202, 191, 11, "f16", "packed"),
    (700, 300, 136, 16, "f16", "paper"), (1025, 260, 200, 6, "f16", "paper"),
    # tiles of 1024 rows x 32 outputs (bfloat16): the smallest batch, odd output counts, every pitch of a grid line
    (256, 600, 260, 16, "bf16", "packed"), (1023, 400, 97, 12, "bf16", "packed"), (1025, 400, 67, 15, "bf16", "packed"),
    (1024, 300, 100, 17, "bf16", "packed"), (2049, 300, 65, 20, "bf16", "packed"), (1100, 300, 100, 30, "bf16", "packed"),
    (1030, 202, 130, 33, "bf16", "packed"), (1030, 202, 130, 34, "bf16", "packed"), (3000, 200, 33, 32, "bf16", "packed")])
def test_grad_x_matches_the_oracle(oracle, B, n_in, n_out, G, storage, layout):
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, layout)
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    assert rowwise_rel_err(_grad_x(desc, x, table, gy), want) <= TOL_F32


@pytest.mark.parametrize("storage,G", [("f16", 16), ("bf16", 16), ("bf16", 24)])
@pytest.mark.parametrize("scale", [1e-30, 1e-8, 1.0, 1e30])
def test_parts_of_gy_hold_every_magnitude(oracle, storage, G, scale):
    """A row is scaled as a whole; within a row 2^-40 ... 1, whose small values the large ones must not swallow:
    half of the rows have small values only in the outputs of one tile."""
    B, n_in, n_out = 600, 300, 200
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    spread = torch.exp2(-40.0 * torch.rand(gy.shape, generator=torch.Generator().manual_seed(6)))
    gy = gy * scale * torch.where(torch.arange(B)[:, None] % 2 == 0, spread, torch.where(torch.arange(n_out)[None, :] < 64, 2.0 ** -40, 1.0))
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    assert rowwise_rel_err(_grad_x(desc, x, table, gy) / scale, want / scale) <= TOL_F32
    # outputs of the first tile alone: their values are all there is
    gy[:, 64:] = 0.0
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    factor = 2.0 ** 20 / scale       # (float32's smallest numbers are not reached by the sums themselves)
    got = _grad_x(desc, x, table, gy)
    if scale > 1e-20:
        assert rowwise_rel_err(got.astype(np.float64) * factor, want * factor) <= TOL_F32


@pytest.mark.parametrize("storage,G", [("f16", 16), ("bf16", 16), ("bf16", 24)])
def test_values_that_are_not_finite_stay_in_their_row(storage, G):
    B, n_in, n_out = 600, 300, 200
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    clean = _grad_x(desc, x, table, gy)
    gy[7, 3], gy[70, 150], gy[71, 199] = float("nan"), float("inf"), -float("inf")
    got = _grad_x(desc, x, table, gy)
    rows = np.array([7, 70, 71])
    assert not np.isfinite(got[rows]).any()
    others = np.setdiff1d(np.arange(B), rows)
    # (the tiles of a row are added in any order)
    assert rowwise_rel_err(got[others], clean[others].astype(np.float64)) <= TOL_F32


def test_an_infinite_gradient_keeps_its_sign_where_the_table_decides_it():
    """gy = inf times corners of opposite signs: the derivative is an infinity, not a NaN."""
    for storage, G in (("f16", 8), ("bf16", 8), ("bf16", 20)):
        B, n_in, n_out = 300, 400, 140
        x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
        # output 5 grows along the first axis: negative below, positive above; flat along the second
        P[:, :, :, 5] = torch.where(torch.arange(G + 1) < G / 2, -1.0, 1.0).to(P.dtype).cuda()[:, None, None]
        table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0]), P)
        x[:] = 0.01 if G % 2 else -0.01      # the cell on the step's lower side: corners -1 and 1
        gy[:] = 0.0
        gy[0, 5] = float("inf")
        got = _grad_x(desc, x, table, gy)
        assert np.isposinf(got[0, 0::2]).all(), (storage, got[0, :4])
