"""The one-launch kernels of small layers and batches against the oracle, at the sizes where they can go
wrong (lanes per row, slots and waves per row, tiles, remainders, the ends of the tensors, the
workgroup's share of the batch), and layers just large enough to stream their table through LDS with
ragged tiles, so that neither family is only tested at the sizes that suit it."""
import numpy as np
import pytest
import torch

import paper_2509_07103_amd as pkg
from paper_2509_07103_amd import workloads as wl
from parity_util import ORACLE_DTYPE, TOL_F32, bits, output_rel_err, pair_slice_rel_err, rowwise_rel_err

pytestmark = pytest.mark.gpu

DT_CODE = {"f32": pkg.LMKAN_F32, "f16": pkg.LMKAN_F16, "bf16": pkg.LMKAN_BF16}

SMALL = [
    # B, n_in, n_out, G
    (1, 512, 300, 16),      # one row: its pairs over many waves, narrow pieces, a last tile of 44 outputs
    (3, 1030, 129, 5),      # 515 pairs: the last chunk of a wave is not full
    (700, 2, 33, 3),        # one pair: a slot takes several rows
    (701, 6, 65, 9),        # three pairs, the second tile of one output
    (1025, 10, 4, 6),       # one lane per row; the coefficient gradient's larger share per thread
    (1024, 12, 5, 7),       # two lanes, and the last batch of the smaller share
    (40000, 4, 16, 8),      # workgroups go on to further rows
    (513, 40, 17, 12),
    (65, 34, 257, 33),      # three tiles of 128 outputs for the coefficient gradient
    (200, 30, 64, 64),      # 4096 cells
    (3000, 16, 12, 40),
]


def _inputs(B, n_in, n_out, G, seed, dev):
    g = torch.Generator(device="cpu").manual_seed(seed)
    x = torch.randn((B, n_in), generator=g) * (1.0 + 4.0 * torch.rand((B, n_in), generator=g) ** 4)
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g) * 0.1
    gy = torch.randn((B, n_out), generator=g)
    return x.to(dev), P.to(dev), gy.to(dev)


def _check(oracle, shape, storage, seed, accumulate=False):
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = shape
    x, P, gy = _inputs(B, n_in, n_out, G, seed, dev)
    paper = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DT_CODE[storage])
    Ps = wl.store(P, storage).contiguous()
    packed = pkg.lmkan_pack(paper, Ps)
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DT_CODE[storage], coef_layout=pkg.LMKAN_LAYOUT_PACKED,
                         flags=pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF if accumulate else 0)
    y = pkg.lmkan_forward(desc, x, packed)
    start = torch.full(paper.coef_shape(), 0.25, device=dev) if accumulate else None
    gx, gP = pkg.lmkan_backward(desc, x, packed, gy, grad_coef=start)
    torch.cuda.synchronize()
    xh, gyh, code = x.cpu().numpy(), gy.cpu().numpy(), ORACLE_DTYPE[storage]
    assert output_rel_err(y.cpu().numpy(), oracle.forward(xh, bits(Ps), G, dtype=code, threads=8)) <= TOL_F32
    assert rowwise_rel_err(gx.cpu().numpy(), oracle.backward_input(xh, bits(Ps), gyh, G, dtype=code, threads=8)) <= TOL_F32
    gPh = gP.cpu().numpy()
    for k in range(0, n_in // 2, max(1, n_in // 16)):
        want = oracle.backward_coef_pair(xh, gyh, G, k)
        if accumulate:
            assert np.abs(gPh[:, :, k, :] - (want + 0.25)).max() <= 2e-5 * max(1.0, np.abs(want).max())
        else:
            assert pair_slice_rel_err(gPh[:, :, k, :], want) <= TOL_F32
            assert np.all(gPh[:, :, k, :][want == 0.0] == 0.0)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", SMALL)
def test_small_shapes_match_the_oracle(oracle, shape, storage):
    _check(oracle, shape, storage, 71)


@pytest.mark.parametrize("shape", [(513, 40, 17, 12), (65, 34, 260, 9)])
def test_small_shapes_accumulate(oracle, shape):
    _check(oracle, shape, "f32", 72, accumulate=True)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(2600, 512, 193, 16), (3000, 300, 300, 16), (5000, 256, 200, 22), (5000, 256, 203, 28),
                                   (5000, 256, 200, 40)])
def test_streamed_tables_match_the_oracle(oracle, shape, storage):
    _check(oracle, shape, storage, 73)


def test_small_coefficient_gradients_repeat_bit_for_bit():
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = 1500, 24, 70, 5
    x, _, gy = _inputs(B, n_in, n_out, G, 74, dev)
    desc = pkg.LayerDesc(n_in, n_out, G)
    runs = [pkg.lmkan_backward(desc, x, None, gy, need_grad_x=False)[1] for _ in range(3)]
    torch.cuda.synchronize()
    assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])


def test_a_forward_call_that_gathers_leaves_the_promise_of_records_harmless(oracle):
    """LMKAN_FLAG_WORKSPACE_HAS_RECORDS on a shape whose forward call writes no records: the backward
    call works them out itself where it needs them."""
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = 12000, 16, 40, 6
    x, P, gy = _inputs(B, n_in, n_out, G, 75, dev)
    desc = pkg.LayerDesc(n_in, n_out, G)
    reuse = pkg.LayerDesc(n_in, n_out, G, flags=pkg.LMKAN_FLAG_WORKSPACE_HAS_RECORDS)
    need = max(pkg.lmkan_workspace_bytes(desc, B, False), pkg.lmkan_workspace_bytes(desc, B, True))
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=dev)
    pkg.lmkan_forward(desc, x, P, workspace=ws)
    gx, gP = pkg.lmkan_backward(reuse, x, P, gy, workspace=ws)
    torch.cuda.synchronize()
    xh, gyh = x.cpu().numpy(), gy.cpu().numpy()
    assert rowwise_rel_err(gx.cpu().numpy(), oracle.backward_input(xh, P.cpu().numpy(), gyh, G)) <= TOL_F32
    for k in range(n_in // 2):
        assert pair_slice_rel_err(gP.cpu().numpy()[:, :, k, :], oracle.backward_coef_pair(xh, gyh, G, k)) <= TOL_F32


@pytest.mark.parametrize("room", [True, False])
@pytest.mark.parametrize("shape", [(9000, 20, 1, 7),     # copies of the pairs, partial gradients
                                   (2000, 700, 1, 8),    # more pairs than a workgroup has lanes for
                                   (40, 6, 1, 5),        # one workgroup
                                   (4096, 130, 1, 16)])  # samples that reach few nodes: atomics
def test_one_output_coefficient_gradient(oracle, shape, room):
    """With and without a workspace, into an existing gradient and over a stale one."""
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = shape
    x, P, gy = _inputs(B, n_in, n_out, G, 76, dev)
    acc = pkg.LayerDesc(n_in, n_out, G, flags=pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF)
    ws = None if room else torch.empty(256, dtype=torch.uint8, device=dev)
    added = torch.full(acc.coef_shape(), 0.5, device=dev)
    pkg.lmkan_backward(acc, x, None, gy, need_grad_x=False, grad_coef=added, workspace=ws)
    over = torch.full(acc.coef_shape(), 9.0, device=dev)
    pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G), x, None, gy, need_grad_x=False, grad_coef=over, workspace=ws)
    torch.cuda.synchronize()
    want = oracle.backward_coef(x.cpu().numpy(), gy.cpu().numpy(), G)
    assert np.abs(over.cpu().numpy() - want).max() <= TOL_F32 * np.abs(want).max()
    assert np.abs(added.cpu().numpy() - (want + 0.5)).max() <= 2e-5 * max(1.0, np.abs(want).max())


@pytest.mark.parametrize("G", [15, 16, 40])     # odd and even rows of cells; both gradients from one walk at 40
@pytest.mark.parametrize("pattern", ["cell", "row", "column", "ends", "gaps"])
def test_walks_that_skip_cells(oracle, pattern, G):
    """Coefficient gradients from the cell-sorted samples, where the walk steps from cell to cell, jumps
    inside a row of cells, from row to row, or sees one cell only."""
    dev = torch.device("cuda:0")
    B, n_in, n_out = 3000, 300, 300
    x, P, gy = _inputs(B, n_in, n_out, G, 77, dev)
    a, b = x[:, 0::2], x[:, 1::2]
    if pattern in ("cell", "column"):
        b.fill_(0.3)
    if pattern in ("cell", "row"):
        a.fill_(-0.2)
    if pattern == "ends":                       # the four corner cells of the grid
        x.copy_(torch.where(x > 0, 9.0, -9.0))
    if pattern == "gaps":                       # a few cells, some of them neighbours
        x.copy_((x * 1.5).round() / 1.5)
    _, gP = pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G), x, P, gy)
    torch.cuda.synchronize()
    xh, gyh, gPh = x.cpu().numpy(), gy.cpu().numpy(), gP.cpu().numpy()
    for k in range(0, n_in // 2, 10):
        want = oracle.backward_coef_pair(xh, gyh, G, k)
        # up to 3000 terms meet in a node and may cancel: the scale of a sum's rounding is that of its magnitudes
        scale = np.abs(oracle.backward_coef_pair(xh, np.abs(gyh), G, k)).max()
        assert np.abs(gPh[:, :, k, :] - want).max() <= TOL_F32 * scale
        assert np.all(gPh[:, :, k, :][want == 0.0] == 0.0)


def test_a_gradient_that_gathers_leaves_the_records_it_promises(oracle):
    """The coefficient gradient alone gathers, the forward pass of the same layer streams slabs: flagged
    calls on the workspace of the first give what calls without the flag give."""
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = 591, 264, 800, 15
    x, P, gy = _inputs(B, n_in, n_out, G, 78, dev)
    paper = pkg.LayerDesc(n_in, n_out, G, coef_dtype=pkg.LMKAN_BF16)
    Ps = wl.store(P, "bf16").contiguous()
    packed = pkg.lmkan_pack(paper, Ps)
    plain, reuse = (pkg.LayerDesc(n_in, n_out, G, coef_dtype=pkg.LMKAN_BF16, coef_layout=pkg.LMKAN_LAYOUT_PACKED, flags=f)
                    for f in (0, pkg.LMKAN_FLAG_WORKSPACE_HAS_RECORDS))
    need = max(pkg.lmkan_workspace_bytes(plain, B, False), pkg.lmkan_workspace_bytes(plain, B, True))
    ws = torch.zeros((need,), dtype=torch.uint8, device=dev)
    pkg.lmkan_backward(plain, x, None, gy, need_grad_x=False, workspace=ws)
    y = pkg.lmkan_forward(reuse, x, packed, workspace=ws)
    gx, _ = pkg.lmkan_backward(reuse, x, packed, gy, need_grad_coef=False, workspace=ws)
    torch.cuda.synchronize()
    xh, gyh, code = x.cpu().numpy(), gy.cpu().numpy(), ORACLE_DTYPE["bf16"]
    assert output_rel_err(y.cpu().numpy(), oracle.forward(xh, bits(Ps), G, dtype=code, threads=8)) <= TOL_F32
    assert rowwise_rel_err(gx.cpu().numpy(), oracle.backward_input(xh, bits(Ps), gyh, G, dtype=code, threads=8)) <= TOL_F32
