"""Weight gradients at the channel counts around the tiles' edges and at piece lengths around the batches' edges (one
pair, a batch, an odd first pair, several offsets with no pair at all), against the oracle."""
import pytest

from oracle import sparse_conv as oc
from workloads import generators as gen
from _util import coords_dev, make_layer, norm_err

pytestmark = pytest.mark.gpu


def _check(c, dtype, c_in, c_out, pieces, seed):
    import paper_2311_12862_amd as sp
    ref = oc.build_kmap(c, 3, 1)
    (x32, x), _, (g32, g) = make_layer(ref.n_in, ref.n_out, c_in, c_out, 27, dtype, seed)
    want = oc.wgrad(x32, g32, ref.M)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    for n in pieces:
        cfg = sp.Config(wgrad_pairs=n) if n else None
        dw = sp.wgrad(x, g, km, cfg)
        assert norm_err(dw, want) <= 1e-4, n
        assert (dw == sp.wgrad(x, g, km, cfg)).all(), n


@pytest.mark.parametrize("c_in,c_out", [(8, 16), (32, 32), (40, 64), (64, 24), (72, 96), (104, 40), (128, 136), (264, 16)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_channels(dtype, c_in, c_out):
    _check(gen.lidar_scene(51, target_n=1200), dtype, c_in, c_out, (0, 1, 31, 33, 129, 4000), c_in)


@pytest.mark.parametrize("n", [1, 2, 33, 700])
@pytest.mark.parametrize("dtype,ch", [("f16", 32), ("bf16", 64), ("f16", 96), ("f16", 160), ("f32", 64)])
def test_few_pairs(dtype, ch, n):
    _check(gen.uniform_cloud(n, max(2, int(round((3 * n) ** (1 / 3)))) + 1, seed=n), dtype, ch, ch, (0, 7), n)


def test_wide_tile():
    """The 256 x 256 tile (it needs half a million pairs to be chosen), ragged in both directions."""
    _check(gen.full_grid(29, 1, seed=6), "bf16", 136, 200, (0,), 3)


@pytest.mark.parametrize("c_in,c_out", [(24, 200), (136, 64), (400, 16), (72, 136)])
def test_uneven_channels_with_many_pairs(c_in, c_out):
    """One narrow side, at the pair counts of the 256 x 256 tile."""
    _check(gen.full_grid(29, 1, seed=7), "f16", c_in, c_out, (0,), c_in)


@pytest.mark.parametrize("c_in,c_out", [(128, 104), (96, 40), (256, 128)])
def test_whole_rounds(c_in, c_out):
    """Pair counts at which the number of pieces goes down to whole rounds of one workgroup per CU, on a build that is
    waited for and on one whose pair count only the device knows."""
    import paper_2311_12862_amd as sp
    c = gen.full_grid(26, 1, seed=8)
    _check(c, "f16", c_in, c_out, (0,), c_in)
    (_, x), _, (_, g) = make_layer(len(c), len(c), c_in, c_out, 27, "f16", c_in)
    known, pending = sp.build_kmap(coords_dev(c), 3, 1), sp.build_kmap(coords_dev(c), 3, 1, asynchronous=True)
    want = sp.wgrad(x, g, known).double().cpu().numpy()
    assert norm_err(sp.wgrad(x, g, pending), want) <= 1e-5
    pending.status()


@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 640, 512), ("bf16", 400, 776), ("f32", 320, 256)])
def test_very_wide_layers(dtype, c_in, c_out):
    _check(gen.lidar_scene(52, target_n=1500), dtype, c_in, c_out, (0, 777), c_in)


@pytest.mark.parametrize("dtype,ch", [("f16", 768), ("f32", 256)])
def test_very_wide_layers_keep_their_pieces_short(dtype, ch):
    """However many tiles a layer has, its longest offset (a quarter of all pairs here) is not left to one workgroup per
    tile: that took two to three times as long as pieces of 4,096 pairs."""
    import torch
    import paper_2311_12862_amd as sp
    from _util import TORCH_DT
    c = gen.lidar_scene(53, target_n=100_000)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    x, g = (torch.randn(len(c), ch, device="cuda").to(TORCH_DT[dtype]) for _ in range(2))
    dw = torch.empty(27, ch, ch, device="cuda")

    def ms(cfg):
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sp.wgrad(x, g, km, cfg, out=dw)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    assert ms(None) <= 1.4 * ms(sp.Config(wgrad_pairs=4096))


@pytest.mark.parametrize("dtype,c_in,c_out", [("f16", 32, 32), ("bf16", 8, 24), ("f16", 24, 16)])
def test_narrow_layers_on_dense_maps(dtype, c_in, c_out):
    """Gradients taken straight from the map, row counts that leave a part of a batch: against the oracle, the same bits every
    time; values that are not finite reach the offsets that have them and no others, as they do over pairs."""
    import torch
    import paper_2311_12862_amd as sp
    c = gen.full_grid(38, 1, seed=9)[:54_321 if c_in == 8 else 54_880]
    ref = oc.build_kmap(c, 3, 1)
    assert (ref.M >= 0).sum() >= 1_200_000
    (x32, x), _, (g32, g) = make_layer(ref.n_in, ref.n_out, c_in, c_out, 27, dtype, c_in)
    km = sp.build_kmap(coords_dev(c), 3, 1)
    dw = sp.wgrad(x, g, km)
    assert norm_err(dw, oc.wgrad(x32, g32, ref.M)) <= 1e-4
    assert torch.equal(dw, sp.wgrad(x, g, km))
    pairs = sp.Config(wgrad_pairs=1024)
    edge = int((ref.M < 0).sum(1).argmax())
    for at, value in ((edge, float("inf")), (edge, float("nan")), (len(c) - 1, float("-inf"))):
        bad = g.clone()
        bad[at, c_out - 1] = value
        got, want = sp.wgrad(x, bad, km), sp.wgrad(x, bad, km, pairs)
        assert torch.equal(torch.isfinite(got), torch.isfinite(want)) and not torch.isfinite(got).all()
        both = torch.isfinite(got)
        assert (got[both] - want[both]).abs().max() <= 1e-4 * want[both].abs().max()


def _dense():
    return gen.full_grid(38, 1, seed=9)


def _sides(km, c_in, c_out, seed):
    (_, x), _, (_, g) = make_layer(km.n_in, km.n_out, c_in, c_out, 27, "f16", seed)
    return x, g


@pytest.mark.parametrize("wide_first", [False, True])
def test_the_build_s_verdict_does_not_change_the_kernel(wide_first):
    """A weight gradient called while an asynchronous build of a dense map is unresolved has the same bits when it is called
    again after spconv_kmap_status; asked for only after that, it has those of a build that was waited for.  So it has after a wider
    layer on the same kmap."""
    import torch
    import paper_2311_12862_amd as sp
    c = coords_dev(_dense())
    waited, early, late = sp.build_kmap(c, 3, 1), sp.build_kmap(c, 3, 1, asynchronous=True), sp.build_kmap(c, 3, 1, asynchronous=True)
    assert waited.n_pairs() >= 1_200_000
    x, g = _sides(waited, 16, 24, 5)
    xw, gw = _sides(waited, 64, 64, 6)
    if wide_first:
        wide = sp.wgrad(xw, gw, early)
    first = sp.wgrad(x, g, early)
    early.status(), late.status()
    assert early.n_pairs() == waited.n_pairs()
    assert torch.equal(first, sp.wgrad(x, g, early))
    if wide_first:
        assert torch.equal(wide, sp.wgrad(xw, gw, early))
        sp.wgrad(xw, gw, late)
    want = sp.wgrad(x, g, waited)
    assert torch.equal(want, sp.wgrad(x, g, late))
    assert norm_err(first, want.double().cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("build", [dict(K=3, stride=2), dict(K=3, stride=3), dict(K=3, stride=1, dilate=True), dict(K=3, stride=2, transposed=True)])
def test_narrow_layers_on_other_dense_maps(build):
    """Maps with other rows on one side than on the other, and maps whose pairs nobody has counted yet: the same bits before and
    after they are, and the sums that the pairs give."""
    import torch
    import paper_2311_12862_amd as sp
    k, stride = build.pop("K"), build.pop("stride")
    c = coords_dev(gen.full_grid(110 if stride == 3 else 74 if stride == 2 else 38, 1, seed=10))
    km = sp.build_kmap(c, k, stride, **build)
    x, g = _sides(km, 24, 16, 7)
    first = sp.wgrad(x, g, km)
    pairs = km.n_pairs()
    assert torch.equal(first, sp.wgrad(x, g, km))
    want = sp.wgrad(x, g, km, sp.Config(wgrad_pairs=2048))
    assert norm_err(first, want.double().cpu().numpy()) <= 1e-5
    assert torch.equal(first, sp.wgrad(x, g, km)) and torch.equal(want, sp.wgrad(x, g, km, sp.Config(wgrad_pairs=2048)))
    if not build.get("transposed"):   # (a fine row has 3.4 coarse neighbours: these stay with the pairs)
        assert pairs >= 1_200_000 and pairs >= 7 * km.n_out
        assert not torch.equal(first, want)   # (another order of the sums: it is the map that was walked)
