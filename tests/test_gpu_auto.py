"""Calls without a configuration: the library's own row order and the tiles loaded straight into LDS, at row and
channel counts around the edges of blocks, tiles, pieces and sorted stretches, against the oracle.  The library sorts
for layers that are wide for the map's size, so small maps are sorted here by very wide ones."""
import numpy as np
import pytest

from oracle import sparse_conv as oc
from workloads import generators as gen
from _util import TOL, coords_dev, make_layer, norm_err

pytestmark = pytest.mark.gpu


def _check(c, K, stride, transposed, dtype, c_in, c_out, calls, seed):
    import paper_2311_12862_amd as sp
    ref = oc.build_kmap(c, K, stride, transposed)
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, c_in, c_out, K ** 3, dtype, seed)
    km = sp.build_kmap(coords_dev(c), K, stride, transposed)
    want_f, want_d = oc.forward(x32, w32, ref.M), oc.dgrad(g32, w32, ref.M, ref.n_in)
    for i in range(calls):
        f, d = sp.fwd(x, w, km), sp.dgrad(g, w, km)
        assert norm_err(f, want_f) <= TOL[dtype], (i, "fwd")
        assert norm_err(d, want_d) <= TOL[dtype], (i, "dgrad")


@pytest.mark.parametrize("n", [1, 15, 17, 257, 2047, 2049, 4100])
@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 512, 512), ("bf16", 264, 136), ("f32", 256, 64)])
def test_row_counts(n, dtype, c_in, c_out):
    c = gen.uniform_cloud(n, max(2, int(round((4 * n) ** (1 / 3)))) + 1, seed=n)
    _check(c, 3, 1, False, dtype, c_in, c_out, 6 if n < 1000 else 3, n)


@pytest.mark.parametrize("n,dtype,c_in,c_out", [(48, "f32", 1024, 1024), (257, "f32", 448, 448), (257, "bf16", 904, 904)])
def test_small_sorted_maps(n, dtype, c_in, c_out):
    """As few rows as the order is made for at these widths."""
    import torch
    import paper_2311_12862_amd as sp
    assert sp.describe_launch(3, n, n, c_in, c_out, {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]).sorted
    c = gen.uniform_cloud(n, max(2, int(round((4 * n) ** (1 / 3)))) + 1, seed=n)
    _check(c, 3, 1, False, dtype, c_in, c_out, 2, n)


@pytest.mark.parametrize("c_in,c_out", [(8, 16), (40, 24), (64, 32), (96, 72), (136, 64), (192, 128), (64, 200), (320, 264)])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_channel_counts(dtype, c_in, c_out):
    c = gen.lidar_scene(41, target_n=2500)
    _check(c, 3, 1, False, dtype, c_in, c_out, 3, c_in)


@pytest.mark.parametrize("K,stride,transposed", [(3, 2, False), (3, 2, True), (2, 2, False), (2, 2, True), (3, 3, False), (1, 1, False)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_other_maps(K, stride, transposed, dtype):
    c = gen.lidar_scene(43, target_n=3000)
    _check(c, K, stride, transposed, dtype, 128, 192, 4, 7)


def test_large_tiles():
    """256 x 256 and 128 x 128 tiles (they need enough rows to be chosen), ragged at both ends."""
    c = gen.full_grid(20, 26, seed=5)[:200_003]
    import paper_2311_12862_amd as sp
    import torch
    km = sp.build_kmap(coords_dev(c), 3, 1)
    for c_in, c_out in ((32, 256), (40, 136), (64, 128)):
        x = torch.randn(len(c), c_in, device="cuda").half()
        w = (torch.randn(27, c_in, c_out, device="cuda") / 20).half()
        cfg = sp.Config(n_split=1, kernel=2, tile_m=64)   # the register-staged kernel
        assert norm_err(sp.fwd(x, w, km), sp.fwd(x, w, km, cfg).double().cpu().numpy()) <= 2e-3
        g = torch.randn(len(c), c_out, device="cuda").half()
        assert norm_err(sp.dgrad(g, w, km), sp.dgrad(g, w, km, cfg).double().cpu().numpy()) <= 2e-3


def test_same_bits_every_time():
    """The same calls on another kmap of the same rows give the same bits (the order is stable, and which K group
    sums a unit depends on the unit alone)."""
    import paper_2311_12862_amd as sp
    c = gen.lidar_scene(47, target_n=6000)
    (_, x), (_, w), _ = make_layer(len(c), len(c), 128, 128, 27, "f16", 3)
    outs = []
    for _ in range(2):
        km = sp.build_kmap(coords_dev(c), 3, 1)
        outs.append([sp.fwd(x, w, km).cpu().numpy() for _ in range(6)])
    assert all(np.array_equal(a, b) for a, b in zip(*outs))
    assert np.array_equal(outs[0][4], outs[0][5])


def _layer_on(sp, km, c_in, c_out, dtype, seed):
    (_, x), (_, w), (_, g) = make_layer(km.n_in, km.n_out, c_in, c_out, 27, dtype, seed)
    return x, w, g


@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 128, 128), ("f16", 64, 64), ("bf16", 40, 96), ("f32", 32, 48)])
def test_bits_do_not_depend_on_what_ran_before(dtype, c_in, c_out):
    """The first call of a layer on a fresh kmap and its calls after many others, some of which sorted the rows, agree
    to the bit: the kernel does not depend on the kmap's history, and its sums not on the order of the rows."""
    import paper_2311_12862_amd as sp
    import torch
    c = gen.lidar_scene(48, target_n=4000)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    x, w, g = _layer_on(sp, km, c_in, c_out, dtype, 3)
    first = sp.fwd(x, w, km), sp.dgrad(g, w, km)
    xw, ww, gw = _layer_on(sp, km, 512, 512, "f16", 4)
    for i in range(8):
        sp.fwd(xw, ww, km)
        assert torch.equal(first[0], sp.fwd(x, w, km)) and torch.equal(first[1], sp.dgrad(g, w, km)), i


def test_nothing_is_sorted_under_capture():
    """A wide layer on a kmap that only a narrow layer has warmed up, captured: the order is not made inside the capture
    (its launches would run at the replays, and an eager call in between would walk an empty one).  Eager calls before
    the first replay and between the replays make and use it, and everything agrees to the bit."""
    import paper_2311_12862_amd as sp
    import torch
    c = gen.lidar_scene(49, target_n=6000)
    fresh = sp.build_kmap(coords_dev(c), 3, 1)
    x, w, g = _layer_on(sp, fresh, 256, 256, "f16", 5)
    want = sp.fwd(x, w, fresh).clone(), sp.dgrad(g, w, fresh).clone()  # (sorted; loads the kernels too)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    xn, wn, gn = _layer_on(sp, km, 16, 16, "f16", 6)
    sp.fwd(xn, wn, km), sp.dgrad(gn, wn, km)
    y, d = torch.zeros_like(want[0]), torch.zeros_like(want[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sp.fwd(x, w, km, out=y)
        sp.dgrad(g, w, km, out=d)
    assert torch.equal(sp.fwd(x, w, km), want[0]) and torch.equal(sp.dgrad(g, w, km), want[1])
    for i in range(4):
        y.zero_(), d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[0]) and torch.equal(d, want[1]), i
        assert torch.equal(sp.fwd(x, w, km), want[0]), i


def test_without_memory_for_the_order():
    """Where the order cannot be allocated the layer runs in map order, with the same bits, and sorts later."""
    import gc
    import paper_2311_12862_amd as sp
    import torch
    gc.collect()
    held, refuse = {}, []

    def alloc(n, stream):
        if refuse:
            refuse.append(n)
            return 0
        t = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
        held[t.data_ptr()] = t
        return t.data_ptr()

    sp.set_allocator(alloc, lambda ptr, stream: held.pop(ptr, None))
    try:
        c = gen.lidar_scene(50, target_n=5000)
        km = sp.build_kmap(coords_dev(c), 3, 1)
        x, w, g = _layer_on(sp, km, 256, 256, "f16", 7)
        refuse.append("start")
        y, d = sp.fwd(x, w, km), sp.dgrad(g, w, km)
        assert len(refuse) > 1
        refuse.clear()
        have = len(held)
        assert torch.equal(y, sp.fwd(x, w, km)) and torch.equal(d, sp.dgrad(g, w, km))
        assert len(held) > have
        torch.cuda.synchronize()
        km.destroy()
        assert not held
    finally:
        refuse.clear()
        gc.collect()
        torch.cuda.synchronize()
        sp.set_allocator(None, None)


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 97, 2049])
@pytest.mark.parametrize("c_in,c_out", [(4, 16), (12, 20), (16, 64), (36, 36), (68, 100)])
def test_fp32_tiles_in_pairs(n, c_in, c_out):
    """fp32 layers of small maps: a workgroup holds two 32-row tiles, whose masks, units and sums are their own (at most 16
    channels, or 16 columns), or eight K groups of a wave each; row counts around their edges (a last workgroup with an empty or a
    partial second tile)."""
    import torch
    import paper_2311_12862_amd as sp
    info = sp.describe_launch(3, n, n, c_in, c_out, torch.float32)
    assert info.tile_m == 64 and info.waves == 8 and info.tile_n == (16 if c_out <= 16 else 32)
    # (two stages of units: 32-row tiles, two of two groups each; 64-row tiles, eight groups)
    slab = 8192
    assert info.lds_bytes == (2 * 4 * (32 + info.tile_n) * 64 + slab if c_in <= 16 else 2 * 8 * (64 + 32) * 64 + slab)
    c = gen.uniform_cloud(n, max(2, int(round((4 * n) ** (1 / 3)))) + 1, seed=n)
    _check(c, 3, 1, False, "f32", c_in, c_out, 1, n)


@pytest.mark.parametrize("n,c_in,c_out,tile_n", [
    (22_001, 20, 36, 32), (20_033, 36, 36, 32), (27_001, 96, 96, 32),  # two 32 x 32 tiles, 128-byte pieces: one, two, three an offset
    (31_009, 40, 72, 64), (48_001, 64, 64, 64), (64_999, 36, 52, 64)])  # 64 x 64, two K groups
def test_fp32_tiles_of_maps_in_between(n, c_in, c_out, tile_n):
    """fp32 maps too large for eight K groups and too small for single ones, all 27 offsets: ragged last tiles and columns, odd and
    even numbers of pieces."""
    import torch
    import paper_2311_12862_amd as sp
    c = gen.lidar_scene(n, target_n=n + 3000)[:n]
    info = sp.describe_launch(3, n, n, c_in, c_out, torch.float32)
    assert len(c) == n and (info.tile_m, info.tile_n, info.waves, info.k_steps) == (64, tile_n, 8, 32)
    _check(c, 3, 1, False, "f32", c_in, c_out, 1, n)


@pytest.mark.parametrize("c_red,c_cols,last,tile,beyond", [
    (64, 64, 24_576, (32, 16), (32, 32)), (256, 256, 24_576, (32, 16), (64, 32)), (512, 512, 14_336, (32, 16), (64, 32)),
    (1024, 256, 36_864, (32, 16), (64, 32)),                                            # eight K groups
    (32, 64, 31_936, (32, 32), (64, 32)), (64, 32, 95_936, (32, 32), (32, 32)), (96, 32, 127_936, (32, 32), (32, 32))])  # pairs
def test_where_fp32_tiles_end(c_red, c_cols, last, tile, beyond):
    """Columns and channels a unit of the tiles on both sides of the lines between them."""
    import torch
    import paper_2311_12862_amd as sp
    a, b = (sp.describe_launch(3, n, n, c_red, c_cols, torch.float32) for n in (last, last + 1))
    assert (a.tile_n, a.k_steps) == tile and (b.tile_n, b.k_steps) == beyond
    assert (a.tile_n, a.k_steps, a.waves) != (b.tile_n, b.k_steps, b.waves)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 1000, 2049])
@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 64, 64), ("bf16", 96, 40), ("f16", 128, 136), ("bf16", 256, 72), ("f16", 264, 264), ("f32", 20, 36),
                                              ("f32", 64, 68)])
def test_groups_of_one_wave(n, dtype, c_in, c_out):
    """Small maps: eight K groups of one wave each, on 64- and 32-row tiles; row counts around them, column tiles that are
    not full, reductions whose pieces do not deal evenly to the groups; the same bits every time."""
    import torch
    import paper_2311_12862_amd as sp
    info = sp.describe_launch(3, n, n, c_in, c_out, {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype])
    assert info.kernel == 2 and info.waves == 8 and info.k_steps == (16 if dtype == "f32" else 32)
    c = gen.uniform_cloud(n, max(2, int(round((4 * n) ** (1 / 3)))) + 1, seed=n)
    _check(c, 3, 1, False, dtype, c_in, c_out, 2, n)


@pytest.mark.parametrize("c_in,c_out", [(256, 256), (136, 72), (96, 96)])
def test_sorted_small_maps_have_the_bits_of_map_order(c_in, c_out):
    """Which group takes a unit depends on the unit alone: 32- and 64-row tiles of one-wave groups, four and eight of them."""
    import torch
    import paper_2311_12862_amd as sp
    c = gen.lidar_scene(53, target_n=30_000 if c_in < 200 else 3500)
    sorted_, plain = sp.build_kmap(coords_dev(c), 3, 1), sp.build_kmap(coords_dev(c), 3, 1)
    x, w, g = _layer_on(sp, sorted_, c_in, c_out, "f16", 3)
    assert sp.describe_launch(3, len(c), len(c), c_in, c_out, torch.float16).sorted
    want = sp.fwd(x, w, sorted_)
    graph, y = torch.cuda.CUDAGraph(), torch.zeros_like(want)
    narrow = _layer_on(sp, plain, 16, 16, "f16", 4)
    sp.fwd(narrow[0], narrow[1], plain)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):   # (nothing is sorted under capture: the same kernel in map order)
        sp.fwd(x, w, plain, out=y)
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(y, want)


@pytest.mark.parametrize("n", [196_609, 199_937])
@pytest.mark.parametrize("c_in,c_out", [(256, 64), (136, 40)])
def test_alternating_halves(n, c_in, c_out):
    """256 x 256 tiles of 64-byte pieces (input gradients of wide layers, reductions that are not whole 128-byte pieces), ragged in
    rows and columns, with row tiles that few offsets and tiles that all offsets reach, against the register-staged kernel."""
    import paper_2311_12862_amd as sp
    import torch
    c = gen.full_grid(20, 26, seed=5)
    c = np.concatenate([c[:n - 3000], np.stack([np.full(3000, 99), np.arange(3000) * 7, np.zeros(3000), np.zeros(3000)], 1)]).astype(np.int32)
    assert sp.describe_launch(3, n, n, c_out, c_in, torch.float16, dgrad=True).tile_m == 256
    km = sp.build_kmap(coords_dev(c), 3, 1)
    w = (torch.randn(27, c_in, c_out, device="cuda") / 20).half()
    g = torch.randn(n, c_out, device="cuda").half()
    want = sp.dgrad(g, w, km, sp.Config(n_split=1, kernel=2, tile_m=64)).double().cpu().numpy()
    got = sp.dgrad(g, w, km)
    assert norm_err(got, want) <= 2e-3
    assert torch.equal(got, sp.dgrad(g, w, km))


@pytest.mark.parametrize("n", [2048, 8191, 16385, 33_000, 132_000, 263_000])
def test_orders_hold_every_row(n):
    """Around the stretches of places, the shares that workgroups write of them, and 256 workgroups that count: every row is in the
    order once (the layers agree with one that walks the map as built)."""
    import paper_2311_12862_amd as sp
    import torch
    c = gen.lidar_scene(50, target_n=n + n // 4)[:n] if n < 50_000 else gen.uniform_cloud(n, 150, seed=n)
    assert len(c) == n
    km = sp.build_kmap(coords_dev(c), 3, 1)
    (_, x), (_, w), (_, g) = make_layer(n, n, ci := 512 if n < 8192 else 128, co := 512 if n < 4100 else 192, 27, "f16", 6)
    assert sp.describe_launch(3, n, n, ci, co, torch.float16).sorted
    cfg = sp.Config(n_split=0, kernel=2, tile_m=64)
    for got, want in ((sp.fwd(x, w, km), sp.fwd(x, w, km, cfg)), (sp.dgrad(g, w, km), sp.dgrad(g, w, km, cfg))):
        assert norm_err(got, want.double().cpu().numpy()) <= 2e-3  # (two roundings to fp16 of equal sums)
