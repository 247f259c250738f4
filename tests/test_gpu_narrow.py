"""Layers that reduce over 8 or 16 channels (several offsets share a matrix instruction) against the oracle: row counts around
the 16-row blocks, offset counts that do not fill the last group, sorted and split maps; K = 5 in one launch."""
import numpy as np
import pytest

from oracle import sparse_conv as oc
from workloads import generators as gen
from _util import TOL, coords_dev, make_layer, norm_err

pytestmark = pytest.mark.gpu


def _cloud(n):
    return gen.uniform_cloud(n, max(2, int(round((4 * n) ** (1 / 3)))) + 1, seed=n)


def _run(sp, c, K, stride, transposed, dtype, c_in, c_out, cfg, seed):
    ref = oc.build_kmap(c, K, stride, transposed)
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, c_in, c_out, K ** 3, dtype, seed)
    km = sp.build_kmap(coords_dev(c), K, stride, transposed)
    assert norm_err(sp.fwd(x, w, km, cfg), oc.forward(x32, w32, ref.M)) <= TOL[dtype]
    assert norm_err(sp.dgrad(g, w, km, cfg), oc.dgrad(g32, w32, ref.M, ref.n_in)) <= TOL[dtype]
    km.destroy()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 257, 4100])
@pytest.mark.parametrize("c_in,c_out", [(8, 8), (8, 72), (16, 16), (16, 40)])
@pytest.mark.parametrize("K", [3, 5])
def test_row_counts(n, c_in, c_out, K):
    import paper_2311_12862_amd as sp
    _run(sp, _cloud(n), K, 1, False, "f16", c_in, c_out, None, n)


@pytest.mark.parametrize("c_in,c_out", [(16, 264), (8, 520), (16, 512), (16, 520), (264, 16), (520, 16)])
def test_planes_of_wide_layers(c_in, c_out):
    """K = 5 in one launch with many column tiles, and on both sides of the width from which 16 channels take a launch per plane."""
    import paper_2311_12862_amd as sp
    _run(sp, _cloud(777), 5, 1, False, "bf16", c_in, c_out, None, c_in)


@pytest.mark.parametrize("K,stride,transposed", [(1, 1, False), (2, 2, False), (2, 2, True), (3, 2, False), (3, 2, True), (3, 1, False)])
@pytest.mark.parametrize("n_split", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("c_in,c_out", [(8, 16), (16, 8)])
def test_maps_and_splits(K, stride, transposed, n_split, c_in, c_out):
    """27 and 8 offsets in groups of four (the last one full or short of one), and parts of a split, which do not share instructions."""
    import paper_2311_12862_amd as sp
    if n_split > K ** 3:
        pytest.skip("more parts than offsets")
    _run(sp, gen.lidar_scene(61, target_n=2100), K, stride, transposed, "bf16", c_in, c_out, sp.Config(n_split=n_split, kernel=1), 5)


def test_weights_that_no_row_uses_stay_out():
    """An offset that no row of the cloud has contributes nothing, whatever its weights are."""
    import paper_2311_12862_amd as sp
    c = _cloud(1000) * np.array([1, 1, 1, 2], np.int32)   # (even z only: no neighbour at dz = -1, +1)
    ref = oc.build_kmap(c, 3, 1)
    (x32, x), (w32, w), _ = make_layer(ref.n_in, ref.n_out, 8, 16, 27, "f16", 9)
    unused = [k for k in range(27) if not (ref.M[:, k] >= 0).any()]
    assert len(unused) >= 9
    want = oc.forward(x32, w32, ref.M)
    w[unused] = float("inf")
    km = sp.build_kmap(coords_dev(c), 3, 1)
    assert norm_err(sp.fwd(x, w, km), want) <= TOL["f16"]


@pytest.mark.parametrize("c_in", [8, 16])
def test_same_bits_sorted_or_not(c_in):
    """Which offsets share an instruction (8 channels) is fixed: a row's sums do not depend on the rows beside it."""
    import torch
    import paper_2311_12862_amd as sp
    c = gen.lidar_scene(62, target_n=5000)
    (_, x), (_, w), _ = make_layer(len(c), len(c), c_in, 32, 27, "f16", 3)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    assert torch.equal(sp.fwd(x, w, km, sp.Config(kernel=1)), sp.fwd(x, w, km, sp.Config(n_split=1, kernel=1)))
