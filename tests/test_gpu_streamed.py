"""The kernels for larger work against the oracle, at layers that reach them (streamed_shapes.py): tables
streamed through LDS, samples sorted by cell."""
import numpy as np
import pytest
import torch

import paper_2509_07103_amd as pkg
from paper_2509_07103_amd import workloads as wl
from parity_util import ORACLE_DTYPE, TOL_F32, bits, output_rel_err, pair_slice_rel_err, rowwise_rel_err
from streamed_shapes import CONV, DRAWN, FAR_ROWS, REPLAYED, SHAPES, WALKS, WHOLE_STREAMS, every_grid

pytestmark = pytest.mark.gpu

DT_CODE = {"f32": pkg.LMKAN_F32, "f16": pkg.LMKAN_F16, "bf16": pkg.LMKAN_BF16}


def _inputs(B, n_in, n_out, G, seed, dev):
    g = torch.Generator(device="cpu").manual_seed(seed)
    x = torch.randn((B, n_in), generator=g) * (1.0 + 4.0 * torch.rand((B, n_in), generator=g) ** 4)
    P = torch.randn((G + 1, G + 1, n_in // 2, n_out), generator=g) * 0.1
    gy = torch.randn((B, n_out), generator=g)
    return x.to(dev), P.to(dev), gy.to(dev)


def _table(P, n_in, n_out, G, storage, layout, flags=0):
    paper = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DT_CODE[storage])
    stored = wl.store(P, storage).contiguous()
    desc = pkg.LayerDesc(n_in, n_out, G, coef_dtype=DT_CODE[storage], coef_layout=layout, flags=flags)
    return desc, stored, pkg.lmkan_pack(paper, stored) if layout == pkg.LMKAN_LAYOUT_PACKED else stored


def _coef_matches(oracle, gP, xh, gyh, G, pairs, base=0.0):
    """Element by element on a sample of pairs.  Up to 20000 terms meet in a node and may cancel: the scale of a
    sum's rounding is that of its magnitudes; added to `base`, it is rounded at base's magnitude, once for every
    run of the stream that adds (eight half units cover the cases here)."""
    for k in range(0, pairs, max(1, pairs // 8)):
        want = oracle.backward_coef_pair(xh, gyh, G, k)
        scale = np.abs(oracle.backward_coef_pair(xh, np.abs(gyh), G, k)).max()
        assert np.abs(gP[:, :, k, :] - (want + base)).max() <= TOL_F32 * scale + 8 * 2.0 ** -24 * abs(base)
        assert np.all(gP[:, :, k, :][want == 0.0] == base)


@pytest.mark.parametrize("B,n_in,n_out,G,storage,layout,grads,accumulate",
                         [(*s[:6], "both", False) for s in SHAPES] + [(*every_grid(G), "both", False) for G in range(3, 49)] + DRAWN)
def test_layers_match_the_oracle(oracle, B, n_in, n_out, G, storage, layout, grads, accumulate):
    dev = torch.device("cuda:0")
    x, P, gy = _inputs(B, n_in, n_out, G, 91, dev)
    flags = pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF if accumulate else 0
    desc, stored, table = _table(P, n_in, n_out, G, storage, layout, flags)
    base = torch.full(desc.coef_shape(), 0.5, device=dev) if accumulate else None
    y = pkg.lmkan_forward(desc, x, table)
    gx, gP = pkg.lmkan_backward(desc, x, table, gy, need_grad_x=grads != "coef", need_grad_coef=grads != "x", grad_coef=base)
    torch.cuda.synchronize()
    xh, gyh, code = x.cpu().numpy(), gy.cpu().numpy(), ORACLE_DTYPE[storage]
    assert output_rel_err(y.cpu().numpy(), oracle.forward(xh, bits(stored), G, dtype=code, threads=8)) <= TOL_F32
    if grads != "coef":
        assert rowwise_rel_err(gx.cpu().numpy(), oracle.backward_input(xh, bits(stored), gyh, G, dtype=code, threads=8)) <= TOL_F32
    if grads != "x":
        _coef_matches(oracle, gP.cpu().numpy(), xh, gyh, G, n_in // 2, 0.5 if accumulate else 0.0)


@pytest.mark.parametrize("n,h,w,c,window,stride,n_out,G,storage,layout", [s[:10] for s in CONV])
def test_convolutions_match_the_oracle(oracle, n, h, w, c, window, stride, n_out, G, storage, layout):
    dev = torch.device("cuda:0")
    n_in = window * window * c
    conv = pkg.Conv2d(n, h, w, c, window, window, stride)
    rows, oh, ow = pkg.lmkan_conv2d_rows(conv)
    _, P, gy = _inputs(rows, n_in, n_out, G, 92, dev)
    x = torch.randn((n, h, w, c), generator=torch.Generator(device="cpu").manual_seed(93)).to(dev)
    desc, stored, table = _table(P, n_in, n_out, G, storage, layout)
    y = pkg.lmkan_conv2d_forward(desc, conv, x, table)
    gx, gP = pkg.lmkan_conv2d_backward(desc, conv, x, table, gy.view(n, oh, ow, n_out))
    torch.cuda.synchronize()
    # the windows as rows, and the rows' gradient summed back into the image
    element = torch.arange(n * h * w * c).view(n, h, w, c)
    rows_of = element.unfold(1, window, stride).unfold(2, window, stride).permute(0, 1, 2, 4, 5, 3).reshape(rows, n_in)
    xh, gyh, code = x.cpu().flatten()[rows_of].numpy(), gy.cpu().numpy(), ORACLE_DTYPE[storage]
    assert output_rel_err(y.cpu().numpy().reshape(rows, n_out), oracle.forward(xh, bits(stored), G, dtype=code, threads=8)) <= TOL_F32
    gx_rows = oracle.backward_input(xh, bits(stored), gyh, G, dtype=code, threads=8)
    want = np.zeros(element.numel())
    np.add.at(want, rows_of.numpy().ravel(), gx_rows.ravel())
    assert rowwise_rel_err(gx.cpu().numpy().reshape(n, -1), want.reshape(n, -1)) <= TOL_F32
    _coef_matches(oracle, gP.cpu().numpy(), xh, gyh, G, n_in // 2)


@pytest.mark.parametrize("B,n_in,n_out,G,storage,layout", [s[:6] for s in SHAPES if "slab" in s[6] or "lane" in s[6]][::3])
def test_calls_reuse_the_records_of_another_call(B, n_in, n_out, G, storage, layout):
    """LMKAN_FLAG_WORKSPACE_HAS_RECORDS after a forward call and after each kind of backward call: what the calls
    without the flag give (the order of float atomics aside)."""
    dev = torch.device("cuda:0")
    x, P, gy = _inputs(B, n_in, n_out, G, 96, dev)
    desc, _, table = _table(P, n_in, n_out, G, storage, layout)
    reuse = pkg.LayerDesc(n_in, n_out, G, coef_dtype=desc.coef_dtype, coef_layout=layout, flags=pkg.LMKAN_FLAG_WORKSPACE_HAS_RECORDS)
    need = max(pkg.lmkan_workspace_bytes(desc, B, False), pkg.lmkan_workspace_bytes(desc, B, True))
    want_y = pkg.lmkan_forward(desc, x, table)
    want_gx, want_gP = pkg.lmkan_backward(desc, x, table, gy)
    fill = [lambda ws: pkg.lmkan_forward(desc, x, table, workspace=ws),
            lambda ws: pkg.lmkan_backward(desc, x, table, gy, need_grad_x=False, workspace=ws),
            lambda ws: pkg.lmkan_backward(desc, x, table, gy, need_grad_coef=False, workspace=ws)]
    for first in fill:
        ws = torch.zeros(need, dtype=torch.uint8, device=dev)
        first(ws)
        gx, gP = pkg.lmkan_backward(reuse, x, table, gy, workspace=ws)
        y = pkg.lmkan_forward(reuse, x, table, workspace=ws)
        torch.cuda.synchronize()
        assert rowwise_rel_err(y.cpu().numpy(), want_y.cpu().numpy().astype(np.float64)) <= 1e-6
        assert rowwise_rel_err(gx.cpu().numpy(), want_gx.cpu().numpy().astype(np.float64)) <= TOL_F32
        assert float((gP - want_gP).abs().max()) <= TOL_F32 * float(want_gP.abs().max())


def test_whole_streams_repeat_bit_for_bit():
    dev = torch.device("cuda:0")
    B, n_in, n_out, G = WHOLE_STREAMS
    x, _, gy = _inputs(B, n_in, n_out, G, 94, dev)
    desc = pkg.LayerDesc(n_in, n_out, G)
    runs = [pkg.lmkan_backward(desc, x, None, gy, need_grad_x=False)[1] for _ in range(3)]
    torch.cuda.synchronize()
    assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])


@pytest.mark.parametrize("B,n_in,n_out,G", WALKS)
def test_input_gradients_of_the_walk_repeat_bit_for_bit(B, n_in, n_out, G):
    dev = torch.device("cuda:0")
    x, P, gy = _inputs(B, n_in, n_out, G, 95, dev)
    desc, _, table = _table(P, n_in, n_out, G, "f32", pkg.LMKAN_LAYOUT_PACKED)
    runs = [pkg.lmkan_backward(desc, x, table, gy)[0] for _ in range(3)]
    torch.cuda.synchronize()
    assert torch.equal(runs[0], runs[1]) and torch.equal(runs[0], runs[2])


@pytest.mark.parametrize("B,n_in,n_out,G,storage,layout", REPLAYED)
def test_replays_of_a_captured_step_match_eager_calls(B, n_in, n_out, G, storage, layout):
    """Records, sort, partial outputs, runs that meet in a cleared gradient: recorded once and replayed on other
    inputs, with eager work and synchronisations between the replays."""
    dev = torch.device("cuda:0")
    x, P, gy = _inputs(B, n_in, n_out, G, 97, dev)
    desc, _, table = _table(P, n_in, n_out, G, storage, layout)
    reuse = pkg.LayerDesc(n_in, n_out, G, coef_dtype=desc.coef_dtype, coef_layout=layout, flags=pkg.LMKAN_FLAG_WORKSPACE_HAS_RECORDS)
    need = max(pkg.lmkan_workspace_bytes(desc, B, False), pkg.lmkan_workspace_bytes(desc, B, True))
    ws = torch.zeros(need, dtype=torch.uint8, device=dev)
    y, gx, gP = torch.empty_like(gy), torch.empty_like(x), torch.empty(desc.coef_shape(), device=dev)

    def step():
        pkg.lmkan_forward(desc, x, table, y=y, workspace=ws)
        pkg.lmkan_backward(reuse, x, table, gy, grad_x=gx, grad_coef=gP, workspace=ws)

    step()                      # kernel attributes are set outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        xs, _, gys = _inputs(B, n_in, n_out, G, 100 + rep, dev)
        y_e = pkg.lmkan_forward(desc, xs, table)
        gx_e, gP_e = pkg.lmkan_backward(desc, xs, table, gys)
        torch.cuda.synchronize()
        x.copy_(xs)
        gy.copy_(gys)
        for t in (y, gx, gP):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_e), rep             # the forward sums in a fixed order
        assert float((gx - gx_e).abs().max()) <= TOL_F32 * float(gx_e.abs().max())
        assert float((gP - gP_e).abs().max()) <= TOL_F32 * float(gP_e.abs().max())


@pytest.mark.parametrize("n_in,n_out,G,storage", FAR_ROWS)
def test_rows_of_a_table_4_gib_apart(n_in, n_out, G, storage):
    """Layout of Alg. 1: outputs and derivatives are those of the layer that has 192 of the outputs alone."""
    torch.cuda.empty_cache()
    gen = torch.Generator(device="cuda").manual_seed(4)
    P = torch.empty((G + 1, G + 1, n_in // 2, n_out), dtype=torch.float16 if storage == "f16" else torch.float32, device="cuda")
    P.uniform_(-0.1, 0.1, generator=gen)
    x, gy = (torch.randn((512, n), device="cuda", generator=gen) for n in (n_in, n_out))
    first = (0, n_out // 128 * 64, n_out - 64)
    few = torch.cat([P.narrow(3, at, 64) for at in first], 3)
    gy_few = torch.cat([gy.narrow(1, at, 64) for at in first], 1)
    gy.zero_()
    for i, at in enumerate(first):
        gy[:, at:at + 64] = gy_few[:, i * 64:i * 64 + 64]
    of = dict(coef_dtype=DT_CODE[storage])
    y = pkg.lmkan_forward(pkg.LayerDesc(n_in, n_out, G, **of), x, P)
    gx, _ = pkg.lmkan_backward(pkg.LayerDesc(n_in, n_out, G, **of), x, P, gy, need_grad_coef=False)
    y_few = pkg.lmkan_forward(pkg.LayerDesc(n_in, 192, G, **of), x, few)
    gx_few, _ = pkg.lmkan_backward(pkg.LayerDesc(n_in, 192, G, **of), x, few, gy_few, need_grad_coef=False)
    y = torch.cat([y.narrow(1, at, 64) for at in first], 1)
    assert rowwise_rel_err(y.cpu().numpy(), y_few.double().cpu().numpy()) <= TOL_F32
    assert rowwise_rel_err(gx.cpu().numpy(), gx_few.double().cpu().numpy()) <= TOL_F32
