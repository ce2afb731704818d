"""Which kernels a call takes, on the host: the library's own dispatch with its launches written down
instead of run (routes.py)."""
import random

import pytest

import paper_2509_07103_amd as pkg
from routes import names, recorder, routes, variants
from streamed_shapes import FAR_ROWS

REUSE = pkg.LMKAN_FLAG_WORKSPACE_HAS_RECORDS

# the kernels that read the preamble records
READERS = {"sort_kernel", "forward_slab_kernel", "forward_slab_f16_kernel", "forward_slab_narrow_kernel",
           "forward_lane32_kernel", "forward_lane32_f32_kernel", "forward_small_kernel",
           "backward_input_slab_kernel", "backward_input_lane_kernel", "backward_input_slab_f16_kernel",
           "backward_input_slab_narrow_kernel", "backward_input_lane32_kernel", "backward_input_lane32_f32_kernel",
           "backward_input_small_kernel", "backward_coef_small_kernel"}     # (backward_fused_kernel: after the sort)
WITHOUT = {"forward_generic_kernel", "forward_gather_kernel", "forward_head_kernel", "backward_generic_kernel",
           "backward_gather_kernel", "backward_input_gather_kernel", "backward_coef_gather_kernel",
           "backward_input_head_kernel", "backward_coef_head_kernel", "backward_coef_stream_kernel",
           "backward_fused_kernel", "preamble_records_kernel"}
AROUND = {"fill_zero_kernel", "clear_shared_nodes_kernel", "gy_tiles_kernel", "transpose_kernel", "sum_partials_kernel", "head_combine_kernel",
          "gx_combine_kernel", "conv_input_gradient_kernel", "conv_input_gradient_scatter_kernel"}


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    return recorder(tmp_path_factory.mktemp("recorder"))


def _layer(rng):
    """A layer and batch anywhere in the range the rules choose from."""
    def log(low, high):
        return round(low * (high / low) ** rng.random())
    return dict(n_in=2 * log(1, 1024), n_out=rng.choice([1, 4, 10, log(1, 1024), log(64, 2048)]),
                grid=rng.choice([rng.randint(3, 16), rng.randint(17, 64)]), batch=log(1, 60000),
                dtype=rng.randint(0, 2), layout=rng.choice([0, 1, 1]))


def _calls(layer, rng):
    """Every way a call may fill the workspace: the passes, as rows and as 1 x 1 windows, buffers that only
    have the alignment of their elements."""
    passes = [dict(fn="forward"), dict(fn="backward"), dict(fn="backward", grad_coef=0), dict(fn="backward", grad_x=0)]
    element = 4 if layer["dtype"] == 0 else 2
    for p in passes:
        yield dict(layer, **p)
        yield dict(layer, **p, conv=(layer["batch"], 1, 1, layer["n_in"], 1, 1, 1))
        yield dict(layer, **p, **{b: 4 for b in ("x", "y", "gy", "gx", "gp") if rng.random() < 0.5},
                   coef=element * rng.randint(0, 1))


def _reads_unwritten_records(first, second):
    return READERS & set(names(second)) and "preamble_records_kernel" not in names(second) + names(first)


def test_a_promise_of_records_is_kept_or_ignored(rec):
    """LMKAN_FLAG_WORKSPACE_HAS_RECORDS after any call that was given the workspace it asked for: either
    that call wrote the records or the flagged call does."""
    rng = random.Random(5)
    # grad_x gathers while the coefficient gradient is sorted; the coefficient gradient gathers while the
    # forward pass and grad_x stream slabs; one output, where the kernels for rows write no records
    layers = [dict(n_in=314, n_out=13, grid=16, batch=50094, dtype=0, layout=1),
              dict(n_in=264, n_out=800, grid=15, batch=591, dtype=2, layout=1),
              dict(n_in=64, n_out=1, grid=16, batch=4000, dtype=0, layout=0),
              dict(n_in=1024, n_out=1024, grid=16, batch=8192, dtype=1, layout=1)]
    layers += [_layer(rng) for _ in range(250)]
    calls, pairs = [], []
    for layer in layers:
        own = list(_calls(layer, rng))
        pairs.append((len(calls), len(own)))
        calls += own + [dict(c, flags=REUSE) for c in own]
    got = routes(calls, rec)
    seen = set()
    for at, n in pairs:
        for i in range(at, at + n):
            status, first = got[i]
            assert status == 0
            seen |= set(names(first))
            for j in range(at + n, at + 2 * n):
                assert not _reads_unwritten_records(first, got[j][1]), (calls[i], calls[j], first, got[j][1])
    assert seen <= READERS | WITHOUT | AROUND, seen - READERS - WITHOUT
    assert READERS <= seen, READERS - seen      # the draw reaches all of them


def test_the_static_scratch_takes_every_batch_whose_records_fit(rec):
    """lmkan_forward_static splits the pairs as far as partial outputs fit its buffer; where all fit, it
    launches what lmkan_forward launches."""
    rng = random.Random(6)
    limit, mib = pkg.LMKAN_STATIC_SCRATCH_BYTES, 1 << 20
    # 1.3 MB of records; the quickest split has 59 MB of partial outputs
    layers = [dict(n_in=48, n_out=3256, grid=30, batch=4698, dtype=2, layout=1),
              dict(n_in=1024, n_out=1024, grid=16, batch=8192, dtype=0, layout=1)]     # 50 MB of records
    layers += [_layer(rng) for _ in range(400)]
    got = routes([dict(layer, fn=fn) for layer in layers for fn in ("workspace", "forward", "forward_static")
                  for layer in [dict(layer, grad_x=0, grad_coef=0, pass_=0)]], rec)
    fewer = 0
    for i, layer in enumerate(layers):
        (size, _), (status, free), (static_status, static) = got[3 * i:3 * i + 3]
        assert status == 0
        records = layer["n_in"] // 2 * layer["batch"] * 12 if size else 0
        assert static_status == (7 if records > limit else 0), layer
        if size <= limit:
            assert static == free
        elif static_status == 0:
            assert names(static)[:2] == names(free)[:2]
            assert static[1][1][0] < free[1][1][0]
            fewer += 1
    assert got[2][0] == 0 and got[5][0] == 7 and fewer >= 3, fewer


def test_one_packed_output_gathers_while_rows_are_few(rec):
    """Rows of a layer with one output: the kernel that keeps the tables in LDS, unless few rows make its
    filling the larger part; windows gather or go the generic way; an unaligned table is none for gathers."""
    def main(batch, n_in=256, grid=16, **more):
        call = dict(dict(n_in=n_in, n_out=1, grid=grid, batch=batch, layout=1, fn="forward"), **more)
        (status, launches), = routes([call], rec)
        assert status == 0
        return [n for n in names(launches) if n != "fill_zero_kernel"]
    for batch in (1, 16, 256):
        assert main(batch) == ["forward_gather_kernel"]
        assert main(batch, coef=4) == ["forward_head_kernel"]
    for batch in (30000, 200000):
        for n_in, grid in ((16, 6), (256, 16), (1000, 8)):
            assert main(batch, n_in, grid) == ["forward_head_kernel"]
    assert main(0, conv=(64, 1, 1, 256, 1, 1, 1)) == ["forward_gather_kernel"]
    assert main(64, layout=0) == ["forward_head_kernel"]


def test_both_gradients_take_no_general_kernel_that_one_alone_does_not(rec):
    """The choices of a call for both gradients depend on each other; none may leave grad_x or the coefficient
    gradient to the generic kernel when a call for that gradient alone has a better one (a million
    multiply-adds and more: below, the generic kernel can be the better one)."""
    rng = random.Random(7)
    layers = [dict(n_in=200, n_out=100, grid=36, batch=400, dtype=1, layout=0),
              dict(n_in=612, n_out=12, grid=50, batch=1613, dtype=2, layout=0)]
    layers += [dict(_layer(rng), layout=rng.randint(0, 1)) for _ in range(600)]
    layers = [layer for layer in layers if layer["n_in"] // 2 * layer["n_out"] * layer["batch"] > 1 << 20]
    calls = [dict(layer, fn="backward", **which) for layer in layers for which in ({}, dict(grad_coef=0), dict(grad_x=0))]
    got = routes(calls, rec)
    for i, layer in enumerate(layers):
        both, alone = names(got[3 * i][1]), names(got[3 * i + 1][1]) + names(got[3 * i + 2][1])
        assert both.count("backward_generic_kernel") <= alone.count("backward_generic_kernel"), (layer, both, alone)


def test_few_outputs_keep_their_kernel_when_the_table_is_not_aligned(rec):
    """A table that starts on its element size only cannot be gathered 16 bytes at a time; up to eight outputs
    where no slab kernel applies then take the kernel that works from the records, as without the gathers."""
    for n_out, layout in ((3, 1), (8, 1), (4, 0), (8, 0)):
        layer = dict(n_in=40, n_out=n_out, grid=40, batch=2000, layout=layout, coef=4)
        calls = [dict(layer, fn="forward"), dict(layer, fn="forward", flags=REUSE), dict(layer, fn="forward", coef=0)]
        a, reuse, aligned = (names(launches) for _, launches in routes(calls, rec))
        assert a[0] == "preamble_records_kernel" and a[-1] == "forward_small_kernel" and reuse == a
        assert aligned == ["forward_gather_kernel"]


DTYPE = {"f32": 0, "f16": 1, "bf16": 2}


def test_streamed_shapes_reach_the_kernels_they_are_listed_for(rec):
    from streamed_shapes import CONV, PACKED, REPLAYED, SHAPES, STREAM, WALK, WALKS, WHOLE_STREAMS, every_grid
    layers = [(dict(n_in=n_in, n_out=n_out, grid=G, batch=B, dtype=DTYPE[storage], layout=layout), fwd, both)
              for B, n_in, n_out, G, storage, layout, fwd, both in SHAPES]
    layers += [(dict(n_in=k * k * c, n_out=n_out, grid=G, dtype=DTYPE[storage], layout=layout, conv=(n, h, w, c, k, k, s)), fwd, both)
               for n, h, w, c, k, s, n_out, G, storage, layout, fwd, both in CONV]
    got = routes([dict(layer, fn=fn) for layer, _, _ in layers for fn in ("forward", "backward")], rec)
    seen = set()
    for i, (layer, fwd, both) in enumerate(layers):
        forward, backward = names(got[2 * i][1]), names(got[2 * i + 1][1])
        assert fwd in forward, (layer, forward)
        assert set(both) <= set(backward), (layer, backward)
        seen |= {launch[0] for launch in got[2 * i][1] + got[2 * i + 1][1]}
    # every form of these kernels, except those for tensors of 4 GB and more
    forms = {f"forward_slab_kernel<{t}, {w}>" for t in ("float, 16, 1, 1", "half, 8, 2, 2", "bf16_t, 8, 2, 2") for w in (0, 17)}
    forms |= {f"forward_slab_narrow_kernel<{t}, {s}>" for t in ("float, 16, 4", "half, 8, 8", "bf16_t, 8, 8") for s in ("true", "false")}
    forms |= {f"backward_input_slab_kernel<{t}, 8, 2, 2, {w}>" for t in ("half", "bf16_t") for w in (0, 17)}
    forms |= {f"backward_input_slab_narrow_kernel<{t}>" for t in ("float, 16, 4", "half, 8, 8", "bf16_t, 8, 8")}
    forms |= {f"backward_fused_kernel<{t}, {gp}, true, {r}>" for t in ("float", "half", "bf16_t") for gp in ("true", "false") for r in ("true", "false")}
    forms |= {"forward_slab_f16_kernel", "forward_lane32_f32_kernel", "forward_lane32_kernel<half>", "forward_lane32_kernel<bf16_t>",
              "backward_input_lane32_f32_kernel", "backward_input_lane32_kernel<half>", "backward_input_lane32_kernel<bf16_t>",
              "backward_input_lane_kernel<float, 0>", "backward_input_lane_kernel<float, 17>",
              "backward_input_slab_f16_kernel<0>", "backward_input_slab_f16_kernel<17>", "backward_coef_stream_kernel<true>",
              "gx_combine_kernel", "gy_tiles_kernel", "sum_partials_kernel", "sort_kernel"}
    assert forms <= seen, forms - seen
    # one wave per (pair, tile): the launch is no larger than that
    B, n_in, n_out, G = WHOLE_STREAMS
    (_, launches), = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, fn="backward", grad_x=0)], rec)
    assert [launch[1][0] for launch in launches if launch[0].startswith(STREAM)] == [n_in // 2 * (n_out // 64)]
    for B, n_in, n_out, G in WALKS:
        (_, launches), = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, layout=PACKED, fn="backward")], rec)
        assert WALK in names(launches)
    # forward pass at every grid, and what is recorded into graphs: a kernel that streams the table
    layers = [every_grid(G) for G in range(3, 49)] + REPLAYED
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, dtype=DTYPE[storage], layout=layout, fn="forward")
                  for B, n_in, n_out, G, storage, layout in layers], rec)
    gathered = [layer for layer, (_, launches) in zip(layers, got) if "forward_gather_kernel" in names(launches)]
    assert len(gathered) <= 2, gathered


@pytest.mark.parametrize("grid,n_in,n_out,dtype,layout", [
    (3, 16384, 16384, 0, 0),     # rows of a table node 0.5 GB apart: three of them within a lane's 32 bits
    (3, 32768, 32768, 0, 0),     # 2.1 GB apart
    (3, 32768, 32768, 0, 1),     # packed: 256 bytes apart
    (17, 8192, 8192, 0, 0),      # sixteen rows per load
    (17, 16384, 16384, 0, 0),
    (40, 16384, 16384, 0, 0),
    (16, 32768, 32768, 1, 0), (30, 16384, 16384, 1, 0), (3, 65536, 32768, 2, 0)]
    + [(G, n_in, n_out, DTYPE[storage], 0) for n_in, n_out, G, storage in FAR_ROWS])
def test_rows_of_any_distance_are_streamed(rec, grid, n_in, n_out, dtype, layout):
    call = dict(n_in=n_in, n_out=n_out, grid=grid, batch=512, dtype=dtype, layout=layout)
    for fn in (dict(fn="forward"), dict(fn="backward", grad_coef=0))[:1 if grid > 34 else 2]:
        (status, launches), = routes([dict(call, **fn)], rec)
        assert status == 0
        assert any("slab" in n or "lane" in n for n in names(launches)), names(launches)


@pytest.mark.parametrize("n_out", [65600, 65601, 1048576])
def test_the_regulariser_of_the_largest_layers_can_be_launched(rec, n_out):
    """A 16-bit table of 138 GB and more has more tiles than one dimension of a launch holds threads for."""
    call = dict(n_in=131070, n_out=n_out, grid=3, batch=1, dtype=1, layout=1, fn="hessian", grad_coef=0)
    (status, launches), = routes([call], rec)
    kernel, grid, threads, _ = launches[-1]
    assert status == 0 and kernel.startswith("hessian_reg_kernel")
    assert grid[0] * threads < 1 << 32 and grid[1] < 1 << 16 and grid[0] * grid[1] == (n_out + 63) // 64 * 65535, grid


def test_tables_of_4_gib_and_more_keep_their_kernel(rec):
    """Layout of Alg. 1, float16: a slab's nodes lie up to the whole table apart, rows that one load brings do not."""
    for grid, n in ((16, 4096), (8, 8192), (16, 2048)):
        call = dict(n_in=n, n_out=n, grid=grid, batch=512, dtype=1, layout=0, fn="backward", grad_coef=0)
        (status, launches), = routes([call], rec)
        assert status == 0 and "backward_input_slab_f16_kernel" in names(launches), names(launches)


def test_grad_x_of_16_bit_tables_reaches_the_kernels_it_is_listed_for(rec):
    from streamed_shapes import INPUT_16BIT, SMOOTH_16BIT, UNUSUAL_16BIT
    listed = INPUT_16BIT + SMOOTH_16BIT + UNUSUAL_16BIT
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, dtype=DTYPE[storage], layout=layout, fn="backward", grad_coef=0)
                  for B, n_in, n_out, G, storage, layout, _ in listed], rec)
    for layer, (_, launches) in zip(listed, got):
        assert layer[-1] in names(launches), (layer, names(launches))


@pytest.mark.parametrize("layer,clears", [
    # two runs and more per stream: what they share; all of it below three million entries and in streams of several blocks
    (dict(n_in=256, n_out=128, grid=16, batch=8192), "clear_shared_nodes_kernel"),
    (dict(n_in=160, n_out=128, grid=16, batch=8192), "fill_zero_kernel"),
    (dict(n_in=256, n_out=128, grid=16, batch=12289), "fill_zero_kernel"),
    (dict(n_in=128, n_out=128, grid=40, batch=8192, layout=1), "clear_shared_nodes_kernel"),        # (the walk, with grad_x)
    (dict(n_in=30, n_out=60, grid=47, batch=6810, dtype=1), "fill_zero_kernel"),
    # a run per stream
    (dict(n_in=1024, n_out=512, grid=16, batch=8192), None)])
@pytest.mark.parametrize("adds", [0, 1])
def test_nodes_that_runs_share_are_cleared_unless_added_to(rec, layer, clears, adds):
    walk = layer["grid"] >= 40
    call = dict(layer, fn="backward", grad_x=int(walk), flags=pkg.LMKAN_FLAG_ACCUMULATE_GRAD_COEF if adds else 0)
    (status, launches), = routes([call], rec)
    walks = names(launches)
    assert status == 0 and ("backward_fused_kernel" if walk else "backward_coef_stream_kernel") in walks, walks
    cleared = {"fill_zero_kernel", "clear_shared_nodes_kernel"} & set(walks)
    assert cleared == ({clears} if clears and not adds else set()), walks


@pytest.mark.parametrize("layer,form", [(dict(n_in=256, n_out=128, grid=16, batch=8192), "false"),
                                        (dict(n_in=500, n_out=333, grid=20, batch=1000), "true")])
def test_shared_nodes_are_cleared_in_the_form_of_the_stream(rec, layer, form):
    """Dense and sparse streams name their cells differently: a kernel for each, no choice at run time."""
    (status, launches), = routes([dict(layer, fn="backward", grad_x=0)], rec)
    assert status == 0 and variants(launches, "clear_shared_nodes_kernel") == [form], launches
    assert variants(launches, "sort_kernel") == ["2" if form == "true" else ""], launches


@pytest.mark.parametrize("form", ["NearF32, 16, 4, true", "float, 16, 4, true"])
def test_the_next_slab_is_brought_near_where_its_lines_are_shared(rec, form):
    from streamed_shapes import NEAR, NOT_NEAR
    shapes = NEAR if form.startswith("Near") else NOT_NEAR
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, layout=1, fn="forward") for B, n_in, n_out, G in shapes], rec)
    for shape, (status, launches) in zip(shapes, got):
        assert status == 0 and variants(launches, "forward_slab_narrow_kernel") == [form], (shape, launches)


def test_tiles_that_share_lines_reach_the_kernels_that_place_them(rec):
    from streamed_shapes import SIDE_BY_SIDE, SIDE_BY_SIDE_BF16
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, layout=layout, fn=fn, grad_coef=0)
                  for B, n_in, n_out, G, layout in SIDE_BY_SIDE for fn in ("forward", "backward")], rec)
    for i, shape in enumerate(SIDE_BY_SIDE):
        (fwd, forward), (bwd, backward) = got[2 * i:2 * i + 2]
        assert fwd == 0 and variants(forward, "forward_slab_narrow_kernel") == ["float, 16, 4, false"], (shape, forward)
        assert bwd == 0 and variants(backward, "backward_input_slab_narrow_kernel") == ["float, 16, 4"], (shape, backward)
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, dtype=2, layout=1, fn="backward", grad_coef=0)
                  for B, n_in, n_out, G in SIDE_BY_SIDE_BF16], rec)
    for shape, (status, launches) in zip(SIDE_BY_SIDE_BF16, got):
        assert status == 0 and variants(launches, "backward_input_lane32_kernel") == ["bf16_t"], (shape, launches)


def test_sparse_streams_are_walked_where_cells_of_a_run_hold_few_samples(rec):
    from streamed_shapes import NOT_SPARSE, SPARSE
    got = routes([dict(n_in=n_in, n_out=n_out, grid=G, batch=B, fn="backward", grad_x=0) for B, n_in, n_out, G in SPARSE + NOT_SPARSE], rec)
    runs = set()
    for shape, (status, launches) in zip(SPARSE + NOT_SPARSE, got):
        n_in, n_out, sparse = shape[1], shape[2], shape in SPARSE
        assert status == 0 and variants(launches, "sort_kernel") == ["2" if sparse else ""], (shape, launches)
        form = f"8, {'false' if n_out % 4 else 'true'}" if sparse else "true"
        assert variants(launches, "backward_coef_stream_kernel") == [form], (shape, launches)
        waves, = [grid[0] for name, grid, _, _ in launches if name.startswith("backward_coef_stream_kernel")]
        runs.add((sparse, waves // (n_in // 2 * ((n_out + 63) // 64))))
    assert {1, 2, 4, 8, 16, 32, 64} <= {n for sparse, n in runs if sparse}, runs


def test_rows_of_gy_in_a_sparse_stream_are_within_32_bit_offsets(rec):
    """The walk of sparse cells adds 32-bit offsets to the tile of gy: no batch whose rows reach further is given to it."""
    rng = random.Random(8)
    layers = [dict(n_in=2 * rng.randint(64, 400), n_out=rng.choice([16, 512, 2040, 2044]), grid=rng.randint(46, 64),
                   batch=round(20000 * 100 ** rng.random())) for _ in range(200)]
    sparse = [layer["batch"] * 4 * layer["n_out"] for layer, (_, launches) in
              zip(layers, routes([dict(layer, fn="backward", grad_x=0) for layer in layers], rec)) if variants(launches, "sort_kernel") == ["2"]]
    assert len(sparse) > 50 and 1 << 30 < max(sparse) < 1 << 32
