"""Input gradient of 16-bit tables against the oracle, float16 (lane per sample) and bfloat16 (matrix cores, gy in
parts): edges of the tiles, magnitudes at the ends of the range, values that are not finite, smooth tables.
Sizes from streamed_shapes.py reach these kernels; the smaller ones are gathered."""
import numpy as np
import pytest
import torch

import paper_2509_07103_amd as pkg
from parity_util import ORACLE_DTYPE, TOL_F32, bits, rowwise_rel_err
from streamed_shapes import INPUT_16BIT, PACKED, SMOOTH_16BIT, UNUSUAL_16BIT

pytestmark = pytest.mark.gpu
DTYPE = {"f16": (pkg.LMKAN_F16, torch.float16), "bf16": (pkg.LMKAN_BF16, torch.bfloat16)}


def _layer(B, n_in, n_out, G, storage, layout, seed=5, P=None):
    gen = torch.Generator(device="cpu").manual_seed(seed)
    x = torch.randn((B, n_in), generator=gen) * 1.5
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=gen) * 0.1 if P is None else P
    P = P.to(DTYPE[storage][1]).cuda()
    gy = torch.randn((B, n_out), generator=gen)
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0])
    if layout in ("packed", PACKED):
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
    (1030, 202, 130, 33, "bf16", "packed"), (1030, 202, 130, 34, "bf16", "packed"), (3000, 200, 33, 32, "bf16", "packed")]
    + [layer[:6] for layer in INPUT_16BIT])
def test_grad_x_matches_the_oracle(oracle, B, n_in, n_out, G, storage, layout):
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, layout)
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    assert rowwise_rel_err(_grad_x(desc, x, table, gy), want) <= TOL_F32


_GATHERED = [(600, 300, 200, 16, "f16"), (600, 300, 200, 16, "bf16"), (600, 300, 200, 24, "bf16")]
_STREAMED = [layer[:5] for layer in UNUSUAL_16BIT]


@pytest.mark.parametrize("B,n_in,n_out,G,storage", _GATHERED + _STREAMED)
@pytest.mark.parametrize("scale", [1e-30, 1e-8, 1.0, 1e30])
def test_parts_of_gy_hold_every_magnitude(oracle, B, n_in, n_out, G, storage, scale):
    """A row is scaled as a whole; within a row 2^-40 ... 1, and small values that large ones beside them must not swallow."""
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    spread = torch.exp2(-40.0 * torch.rand(gy.shape, generator=torch.Generator().manual_seed(6)))
    gy = gy * scale * torch.where(torch.arange(B)[:, None] % 2 == 0, spread, torch.where(torch.arange(n_out)[None, :] < 64, 2.0 ** -40, 1.0))
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    assert rowwise_rel_err(_grad_x(desc, x, table, gy) / scale, want / scale) <= TOL_F32
    # small values beside large ones in every tile, whose outputs have a table of zeros: the small ones are all there is
    small = 2.0 ** (-40 if scale > 1e-20 else -6)        # (products stay normal numbers)
    x, P, _, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    P[..., 1::2] = 0.0
    gy[:, 0::2] *= small
    gy *= scale
    table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0]), P)
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8) / (scale * small)
    assert rowwise_rel_err(_grad_x(desc, x, table, gy).astype(np.float64) / (scale * small), want) <= TOL_F32


@pytest.mark.parametrize("B,n_in,n_out,G,storage", _GATHERED + _STREAMED)
def test_values_that_are_not_finite_stay_in_their_row(B, n_in, n_out, G, storage):
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
    gathered = [(300, 400, 140, G, storage) for storage, G in (("f16", 8), ("bf16", 8), ("bf16", 20))]
    for B, n_in, n_out, G, storage in gathered + _STREAMED:
        x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
        # output 5 grows along the first axis: negative below, positive above; flat along the second
        P[:, :, :, 5] = torch.where(torch.arange(G + 1) < G / 2, -1.0, 1.0).to(P.dtype).cuda()[:, None, None]
        table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0]), P)
        x[:] = 0.01 if G % 2 else -0.01      # the cell on the step's lower side: corners -1 and 1
        gy[:] = 0.0
        gy[0, 5] = float("inf")
        got = _grad_x(desc, x, table, gy)
        assert np.isposinf(got[0, 0::2]).all(), (storage, got[0, :4])


# A derivative is a difference of two corners' sums over the outputs.  Summed in float32 over m outputs before it is
# subtracted, term by term, a corner's sum of products p has the error sigma = rho sqrt(sum over r <= m of r var p + r^2 mean^2 p),
# rho = 0.42 2^-24 (root mean square of a relative rounding error over a binade).  On corners that differ by d the
# derivative is d |p| sqrt(2 m) per m outputs, its error sqrt(2) sigma: relative error sigma / (d |p| sqrt m).
def _rounding_bound(m, d, mean_share):
    """mean_share: mean(p)^2 / mean(p^2)."""
    r = np.arange(1, m + 1)
    return 0.42 * 2.0 ** -24 / d * np.sqrt((r * (1 - mean_share) + r * r * mean_share).sum() / m)


@pytest.mark.parametrize("B,n_in,n_out,G,storage,layout", [layer[:6] for layer in SMOOTH_16BIT])
@pytest.mark.parametrize("one_sign", [False, True])
def test_smooth_tables_lose_no_more_than_short_sums_lose(oracle, B, n_in, n_out, G, storage, layout, one_sign):
    """Corners 2 % apart: rounding of the sums of four outputs, and a fifth, is all that may be lost."""
    gen = torch.Generator().manual_seed(9)
    noise = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=gen)
    level = torch.ones((n_in // 2, n_out)) if one_sign else torch.randn((n_in // 2, n_out), generator=gen)
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, layout, P=0.3 * level * (1 + 0.02 * noise))
    gy = gy.abs() if one_sign else gy
    got = _grad_x(desc, x, table, gy)
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert err <= 1.2 * _rounding_bound(4, 0.02, 2 / np.pi if one_sign else 0.0), err


@pytest.mark.parametrize("B,n_in,n_out,G,storage", _STREAMED)
def test_the_largest_finite_gradients(oracle, B, n_in, n_out, G, storage):
    """The sum of a row's |gy| overflows, each of them and every derivative is finite."""
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    P = (P.float() * 2.0 ** -8).to(P.dtype)
    table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0]), P)
    gy = gy.clamp(-3, 3) * 1e38
    want = oracle.backward_input(x.numpy(), bits(P), gy.numpy(), G, dtype=ORACLE_DTYPE[storage], threads=8)
    assert np.abs(want).max() < 3e38
    assert rowwise_rel_err(_grad_x(desc, x, table, gy).astype(np.float64) * 1e-38, want * 1e-38) <= TOL_F32


@pytest.mark.parametrize("B,n_in,n_out,G,storage", _STREAMED)
def test_an_infinite_entry_gives_infinite_derivatives(B, n_in, n_out, G, storage):
    """One node of one pair and output is infinite: the two derivatives of a row in a cell at that node are
    infinities of their signs, all others as they were."""
    cell = (G // 2, G // 2 - 1)
    x, P, table, gy, desc = _layer(B, n_in, n_out, G, storage, "packed")
    nodes = torch.from_numpy(pkg.lmkan_grid(G)[0])
    rows, pair, output = torch.tensor([3, 300, 599]), 7, 150
    middle = [(nodes[c] + nodes[c + 1]) / 2 for c in cell]
    x[:, 2 * pair] = nodes[cell[0] - 2]                    # everyone else is in another column of cells
    x[rows, 2 * pair], x[rows, 2 * pair + 1] = middle[0], middle[1]
    clean = _grad_x(desc, x, table, gy)
    P[cell[0] + 1, cell[1], pair, output] = float("inf")   # the cell's corner 10
    table = pkg.lmkan_pack(pkg.LayerDesc(n_in, n_out, G, coef_dtype=DTYPE[storage][0]), P)
    got = _grad_x(desc, x, table, gy)
    sign = np.sign(gy[rows, output].numpy())
    np.testing.assert_array_equal(got[rows, 2 * pair], sign * np.inf)
    np.testing.assert_array_equal(got[rows, 2 * pair + 1], -sign * np.inf)
    got[rows, 2 * pair], got[rows, 2 * pair + 1] = clean[rows, 2 * pair], clean[rows, 2 * pair + 1]
    assert rowwise_rel_err(got, clean.astype(np.float64)) <= TOL_F32


def test_nodes_more_than_4_gib_apart():
    """Layout of Alg. 1, 4.8 GB: the same derivatives as from the packed table."""
    B, n, G = 300, 4096, 16
    gen = torch.Generator(device="cuda").manual_seed(4)
    P = torch.empty((G + 1, G + 1, n // 2, n), dtype=torch.float16, device="cuda")
    P.uniform_(-0.1, 0.1, generator=gen)
    x, gy = (torch.randn((B, n), device="cuda", generator=gen) for _ in range(2))
    paper = pkg.LayerDesc(n, n, G, coef_dtype=pkg.LMKAN_F16)
    packed = pkg.LayerDesc(n, n, G, coef_dtype=pkg.LMKAN_F16, coef_layout=pkg.LMKAN_LAYOUT_PACKED)
    got, _ = pkg.lmkan_backward(paper, x, P, gy, need_grad_coef=False)
    want, _ = pkg.lmkan_backward(packed, x, pkg.lmkan_pack(paper, P), gy, need_grad_coef=False)
    assert rowwise_rel_err(got.cpu().numpy(), want.double().cpu().numpy()) <= TOL_F32
