"""Kernel maps built by the HIP library against the oracle: bit-exact."""
import numpy as np
import pytest
import torch

from oracle import sparse_conv as oc
from workloads import generators as gen
from _util import coords_dev, make_layer, norm_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_2311_12862_amd as sp
    return sp


def _check_kmap(sp, c, K, stride, transposed):
    ref = oc.build_kmap(c, K, stride, transposed)
    km = sp.build_kmap(coords_dev(c), K, stride, transposed)
    assert (km.n_in, km.n_out) == (ref.n_in, ref.n_out)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.out_coords().cpu().numpy(), ref.out_coords)
    np.testing.assert_array_equal(km.in_coords().cpu().numpy(), ref.in_coords)
    mask = km.export_mask().cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(mask, oc.bitmask(ref.M))
    assert km.n_pairs() == int((ref.M >= 0).sum())
    km.destroy()
    return ref


@pytest.mark.parametrize("n,grid,lo", [(2000, 64, 0), (3000, 16, -8), (700, 9, 100)])
def test_submanifold(sp, n, grid, lo):
    c = gen.uniform_cloud(n, grid, seed=n, lo=lo)
    c[: n // 3, 0] = 2
    _check_kmap(sp, c, 3, 1, False)


@pytest.mark.parametrize("stride", [2, 3])
@pytest.mark.parametrize("lo", [0, -7])
def test_strided(sp, stride, lo):
    c = gen.uniform_cloud(4000, 20, seed=17 + stride, lo=lo)
    c[:1500, 0] = 1
    ref = _check_kmap(sp, c, 3, stride, False)
    assert ref.n_out < 4000


@pytest.mark.parametrize("transposed", [False, True])
def test_even_kernel_stride2(sp, transposed):
    """K = s = 2: the non-overlapping 2x2x2 layer and its transposed counterpart (8 offsets)."""
    c = gen.uniform_cloud(4000, 20, seed=29, lo=-6)
    c[:1300, 0] = 1
    ref = _check_kmap(sp, c, 2, 2, transposed)
    assert ref.M.shape[1] == 8
    _check_kmap(sp, gen.lidar_scene(31, target_n=30_000), 2, 2, transposed)
    _check_kmap(sp, np.array([[0, -1, 0, 3]], dtype=np.int32), 2, 2, transposed)
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(c), 2, 1, transposed)   # the even kernel exists for stride 2 only
    assert e.value.status == -1


@pytest.mark.parametrize("stride", [1, 2])
def test_transposed(sp, stride):
    c = gen.uniform_cloud(3500, 18, seed=23, lo=-5)
    c[:1000, 0] = 3
    _check_kmap(sp, c, 3, stride, True)


def test_k1(sp):
    c = gen.uniform_cloud(1000, 12, seed=5)
    _check_kmap(sp, c, 1, 1, False)
    _check_kmap(sp, c, 1, 2, False)


def test_lidar_scene_small(sp):
    c = gen.lidar_scene(2000, target_n=20_000)
    _check_kmap(sp, c, 3, 1, False)
    _check_kmap(sp, c, 3, 2, False)


def test_empty_single_and_limits(sp):
    km = sp.build_kmap(torch.empty((0, 4), dtype=torch.int32, device="cuda"), 3, 1)
    assert (km.n_in, km.n_out, km.n_pairs()) == (0, 0, 0)
    assert km.export().shape == (0, 27)
    km.destroy()
    _check_kmap(sp, np.array([[0, 5, -3, 7]], dtype=np.int32), 3, 1, False)
    _check_kmap(sp, np.array([[0, 5, -3, 7]], dtype=np.int32), 3, 2, False)
    lim = np.array([[65534, 32767, 32767, 32767], [65534, 32766, 32767, 32766], [0, -32768, -32768, -32768],
                    [0, -32767, -32768, -32768], [0, -32768, 32767, 0]], dtype=np.int32)
    _check_kmap(sp, lim, 3, 1, False)
    _check_kmap(sp, lim, 3, 2, False)
    _check_kmap(sp, lim, 3, 2, True)


def test_errors(sp):
    c = gen.uniform_cloud(500, 10, seed=1)
    dup = c.copy()
    dup[100] = dup[400]
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(dup), 3, 1)
    assert e.value.status == -3
    with pytest.raises(ValueError):
        oc.build_kmap(dup, 3, 1)
    # duplicates and range errors are reported by every kind of build
    for stride, transposed in ((2, False), (3, False), (2, True), (1, True)):
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(dup), 3, stride, transposed)
        assert e.value.status == -3, (stride, transposed)
    r = c.copy()
    r[7] = [0, 32768, 0, 0]
    for stride, transposed in ((2, False), (2, True)):
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(r), 3, stride, transposed)
        assert e.value.status == -2, (stride, transposed)
    for bad in ([0, 32768, 0, 0], [0, 0, -32769, 0], [65535, 0, 0, 0], [-1, 0, 0, 0]):
        r = c.copy()
        r[7] = bad
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(r), 3, 1)
        assert e.value.status == -2
    for K, stride in ((2, 1), (5, 2), (7, 1), (3, 0), (3, 65)):
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(c), K, stride)
        assert e.value.status == -1
    # the library still works after the error paths
    _check_kmap(sp, c, 3, 1, False)


def test_planar_and_line_sets(sp):
    """Degenerate sets (constant z, constant y and z) load one slot class of the hash table."""
    rng = np.random.default_rng(5)
    xy = rng.permutation(90 * 90)[:5000]
    plane = np.stack([np.zeros(5000, np.int64), xy // 90, xy % 90, np.full(5000, 8)], axis=1).astype(np.int32)
    _check_kmap(sp, plane, 3, 1, False)
    _check_kmap(sp, plane, 3, 2, False)
    line = np.stack([np.zeros(3000, np.int64), rng.permutation(6000)[:3000] - 3000, np.full(3000, -4),
                     np.full(3000, 12)], axis=1).astype(np.int32)
    _check_kmap(sp, line, 3, 1, False)
    _check_kmap(sp, line, 3, 2, True)


def test_build_is_deterministic(sp):
    c = gen.uniform_cloud(5000, 24, seed=9)
    a = sp.build_kmap(coords_dev(c), 3, 2)
    b = sp.build_kmap(coords_dev(c), 3, 2)
    assert torch.equal(a.export(), b.export())
    assert torch.equal(a.out_coords(), b.out_coords())


def test_asynchronous_build(sp):
    """spconv_build_kmap_async returns at once; errors and the pair count arrive with spconv_kmap_status."""
    c = gen.lidar_scene(11, target_n=6000)
    ref = oc.build_kmap(c, 3, 1)
    km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=True)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32), oc.bitmask(ref.M))
    km.status()
    assert km.n_pairs() == int((ref.M >= 0).sum())
    dup = c.copy()
    dup[5] = dup[77]
    km = sp.build_kmap(coords_dev(dup), 3, 1, asynchronous=True)
    with pytest.raises(sp.SpconvError) as e:
        km.status()
    assert e.value.status == -3
    with pytest.raises(sp.SpconvError) as e:   # the verdict stays with the kmap
        km.status()
    assert e.value.status == -3
    # calls that resolve the pending build on their own (pair count, executed MACs, tuner) do not swallow it
    import torch
    for resolve in (lambda k: k.n_pairs(), lambda k: k.mac_units(sp.OP_FWD),
                    lambda k: sp.tune(k, 16, 16, torch.float16, sp.OP_WGRAD, 1)):
        km = sp.build_kmap(coords_dev(dup), 3, 1, asynchronous=True)
        resolve(km)
        with pytest.raises(sp.SpconvError) as e:
            km.status()
        assert e.value.status == -3
    bad = c.copy()
    bad[9, 2] = 40000
    km = sp.build_kmap(coords_dev(bad), 3, 1, asynchronous=True)
    with pytest.raises(sp.SpconvError) as e:
        km.status()
    assert e.value.status == -2
    # map kinds without an asynchronous path are built synchronously by the same call
    km = sp.build_kmap(coords_dev(c), 3, 2, asynchronous=True)
    np.testing.assert_array_equal(km.export().cpu().numpy(), oc.build_kmap(c, 3, 2).M)


def test_caller_allocator_backs_every_device_allocation(sp):
    """spconv_set_allocator: with PyTorch's caching allocator installed, builds, plans and
    kernels run out of its blocks, results do not change, and every block comes back."""
    import torch
    from _util import TOL, make_layer, norm_err
    c = gen.lidar_scene(91, target_n=3000)
    ref = oc.build_kmap(c, 3, 2)
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, 32, 64, 27, "f16", 92)
    live, calls = {}, [0, 0]

    def alloc(n, stream):
        t = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        calls[0] += 1
        return t.data_ptr()

    def free(ptr, stream):
        calls[1] += 1
        live.pop(ptr)

    sp.set_allocator(alloc, free)
    try:
        km = sp.build_kmap(coords_dev(c), 3, 2)
        np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
        cfg = sp.Config()
        cfg.n_split, cfg.kernel = 2, 2                     # sorted plan and split partial sums
        assert norm_err(sp.fwd(x, w, km, cfg), oc.forward(x32, w32, ref.M)) <= TOL["f16"]
        assert norm_err(sp.dgrad(g, w, km), oc.dgrad(g32, w32, ref.M, ref.n_in)) <= TOL["f16"]
        assert norm_err(sp.wgrad(x, g, km), oc.wgrad(x32, g32, ref.M)) <= 1e-4
        assert calls[0] > 5 and live
        torch.cuda.synchronize()
        km.destroy()
        assert not live and calls[0] == calls[1]
    finally:
        sp.set_allocator(None, None)
    km = sp.build_kmap(coords_dev(c), 3, 2)                # the library's own pool serves again
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)


def test_stream_ordered_allocator_on_a_side_stream(sp):
    """The allocator callbacks receive the stream of the call in progress.  A stream-ordered
    caching allocator (PyTorch's, which only reuses a block on the stream it was allocated on)
    backs a kmap that lives entirely on a non-default stream: every callback names that stream,
    results match the oracle, and every block comes back."""
    import torch
    from _util import TOL, make_layer, norm_err
    c = gen.lidar_scene(95, target_n=3000)
    ref = oc.build_kmap(c, 3, 2)
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, 32, 64, 27, "f16", 96)
    side = torch.cuda.Stream()
    live, seen = {}, set()

    def alloc(n, stream):
        seen.add(stream)
        with torch.cuda.stream(torch.cuda.ExternalStream(stream) if stream else torch.cuda.default_stream()):
            t = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")   # the caching allocator files it under that stream
        live[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, stream):
        seen.add(stream)
        live.pop(ptr)        # back to the allocator's pool of the stream it was allocated on

    coords = coords_dev(c)
    torch.cuda.synchronize()
    sp.set_allocator(alloc, free)
    try:
        with torch.cuda.stream(side):
            for rep in range(3):                            # blocks are recycled between the rounds
                km = sp.build_kmap(coords, 3, 2)
                cfg = sp.Config()
                cfg.n_split, cfg.kernel = 2, 1 + rep % 2
                y = sp.fwd(x, w, km, cfg)
                dx = sp.dgrad(g, w, km, cfg)
                dw = sp.wgrad(x, g, km)
                m = km.export()
                km.destroy()
                side.synchronize()
                np.testing.assert_array_equal(m.cpu().numpy(), ref.M)
                assert norm_err(y, oc.forward(x32, w32, ref.M)) <= TOL["f16"]
                assert norm_err(dx, oc.dgrad(g32, w32, ref.M, ref.n_in)) <= TOL["f16"]
                assert norm_err(dw, oc.wgrad(x32, g32, ref.M)) <= 1e-4
                assert not live
        assert seen == {side.cuda_stream}
    finally:
        sp.set_allocator(None, None)


@pytest.mark.parametrize("K,stride", [(3, 2), (2, 2), (3, 1), (3, 3), (1, 1)])
def test_transpose_equals_transposed_build(sp, K, stride):
    """spconv_kmap_transpose: the paired transposed convolution's kmap, derived without a rebuild,
    is bit for bit what a build with `transposed` flipped returns (and what the oracle defines)."""
    from _util import TOL, make_layer, norm_err
    c = gen.lidar_scene(93, target_n=2600)
    ref = oc.build_kmap(c, K, stride, False)
    ref_t = oc.build_kmap(c, K, stride, True)
    km = sp.build_kmap(coords_dev(c), K, stride)
    kt = km.transpose()
    assert (kt.n_in, kt.n_out) == (ref_t.n_in, ref_t.n_out) == (km.n_out, km.n_in)
    assert kt.n_pairs() == km.n_pairs() == int((ref.M >= 0).sum())
    np.testing.assert_array_equal(kt.export().cpu().numpy(), ref_t.M)
    direct = sp.build_kmap(coords_dev(c), K, stride, transposed=True)
    np.testing.assert_array_equal(kt.export_mask().cpu().numpy(), direct.export_mask().cpu().numpy())
    np.testing.assert_array_equal(kt.out_coords().cpu().numpy(), direct.out_coords().cpu().numpy())
    np.testing.assert_array_equal(kt.in_coords().cpu().numpy(), direct.in_coords().cpu().numpy())
    # the derived kmap runs every operator, under sorted plans as well
    (x32, x), (w32, w), (g32, g) = make_layer(ref_t.n_in, ref_t.n_out, 32, 16, K ** 3, "f16", 94)
    cfg = sp.Config()
    cfg.n_split = 1
    assert norm_err(sp.fwd(x, w, kt, cfg), oc.forward(x32, w32, ref_t.M)) <= TOL["f16"]
    assert norm_err(sp.dgrad(g, w, kt, cfg), oc.dgrad(g32, w32, ref_t.M, ref_t.n_in)) <= TOL["f16"]
    assert norm_err(sp.wgrad(x, g, kt), oc.wgrad(x32, g32, ref_t.M)) <= 1e-4
    # and transposing twice gives the original structure back (also from a transposed build)
    np.testing.assert_array_equal(kt.transpose().export().cpu().numpy(), ref.M)
    back = direct.transpose()
    np.testing.assert_array_equal(back.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(back.out_coords().cpu().numpy(), km.out_coords().cpu().numpy())
    np.testing.assert_array_equal(back.in_coords().cpu().numpy(), km.in_coords().cpu().numpy())


def test_transpose_of_empty_and_pending_builds(sp):
    import torch
    empty = sp.build_kmap(torch.zeros((0, 4), dtype=torch.int32, device="cuda"), 3, 2)
    t = empty.transpose()
    assert (t.n_in, t.n_out) == (0, 0)
    c = gen.lidar_scene(95, target_n=1500)
    ref_t = oc.build_kmap(c, 3, 1, True)
    km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=True)
    np.testing.assert_array_equal(km.transpose().export().cpu().numpy(), ref_t.M)   # resolves the build first
    dup = np.vstack([c, c[:1]])
    bad = sp.build_kmap(coords_dev(dup), 3, 1, asynchronous=True)
    with pytest.raises(sp.SpconvError) as e:
        bad.transpose()
    assert e.value.status == -3          # SPCONV_EDUP


@pytest.mark.parametrize("stride,transposed", [(1, False), (1, True), (2, False), (2, True), (3, False)])
def test_pointwise_equals_a_k1_build(sp, stride, transposed):
    """spconv_kmap_pointwise: the K = 1 kmap over either row set of a kmap is what a K = 1 build on
    those rows returns (map, mask, coordinates, sizes), and a 1x1x1 layer through it is X . W[0]."""
    import torch
    from _util import make_layer, norm_err, TOL
    c = gen.lidar_scene(96, target_n=2200)
    ref = oc.build_kmap(c, 3, stride, transposed)
    km = sp.build_kmap(coords_dev(c), 3, stride, transposed)
    for on_outputs, rows_ref in ((False, ref.in_coords), (True, ref.out_coords)):
        one_ref = oc.build_kmap(rows_ref, 1, 1)
        got = km.pointwise(on_outputs)
        want = sp.build_kmap(coords_dev(rows_ref), 1, 1)
        assert (got.n_in, got.n_out, got.n_pairs()) == (one_ref.n_in, one_ref.n_out, len(rows_ref))
        np.testing.assert_array_equal(got.export().cpu().numpy(), one_ref.M)
        np.testing.assert_array_equal(got.export().cpu().numpy(), want.export().cpu().numpy())
        np.testing.assert_array_equal(got.export_mask().cpu().numpy(), want.export_mask().cpu().numpy())
        np.testing.assert_array_equal(got.out_coords().cpu().numpy(), rows_ref)
        (x32, x), (w32, w), (g32, g) = make_layer(one_ref.n_in, one_ref.n_out, 32, 48, 1, "f16", 61)
        assert norm_err(sp.fwd(x, w, got), x32.astype(np.float64) @ w32[0].astype(np.float64)) <= TOL["f16"]
        assert norm_err(sp.dgrad(g, w, got), oc.dgrad(g32, w32, one_ref.M, one_ref.n_in)) <= TOL["f16"]
        assert norm_err(sp.wgrad(x, g, got), oc.wgrad(x32, g32, one_ref.M)) <= 1e-4


def test_pointwise_of_empty_and_pending_builds(sp):
    import torch
    empty = sp.build_kmap(torch.zeros((0, 4), dtype=torch.int32, device="cuda"), 3, 1)
    one = empty.pointwise()
    assert (one.n_in, one.n_out, one.n_pairs()) == (0, 0, 0)
    c = gen.lidar_scene(97, target_n=1500)
    km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=True)
    np.testing.assert_array_equal(km.pointwise().export().cpu().numpy(), np.arange(len(c), dtype=np.int32)[:, None])
    bad = sp.build_kmap(coords_dev(np.vstack([c, c[:1]])), 3, 1, asynchronous=True)
    with pytest.raises(sp.SpconvError) as e:
        bad.pointwise()
    assert e.value.status == -3          # SPCONV_EDUP


def test_transposed_partner_outlives_its_source(sp):
    """A kmap and its transpose share their tables by reference count: either may be destroyed
    first, and dropping the source's plans leaves the partner's map intact."""
    c = gen.lidar_scene(98, target_n=1800)
    ref_t = oc.build_kmap(c, 3, 2, True)
    down = sp.build_kmap(coords_dev(c), 3, 2)
    up = down.transpose()
    down.drop_plans()
    np.testing.assert_array_equal(up.export().cpu().numpy(), ref_t.M)
    down.destroy()
    np.testing.assert_array_equal(up.export().cpu().numpy(), ref_t.M)
    np.testing.assert_array_equal(up.out_coords().cpu().numpy(), ref_t.out_coords)
    again = up.transpose()          # back to the strided map, from the partner alone
    np.testing.assert_array_equal(again.export().cpu().numpy(), oc.build_kmap(c, 3, 2).M)
    up.destroy()
    np.testing.assert_array_equal(again.export().cpu().numpy(), oc.build_kmap(c, 3, 2).M)


@pytest.mark.parametrize("seed,n", [(51, 40), (52, 3000)])
def test_dilated_stride1_output_set(sp, seed, n):
    """spconv_build_kmap_dilated: P_out = every point with an input in its neighbourhood (Eq. 1 with
    P_out != P_in).  Output set, map and masks bit-exact against the oracle; features within tolerance."""
    import torch
    from _util import TOL, make_layer, norm_err
    c = gen.lidar_scene(seed, target_n=n) if n > 100 else gen.uniform_cloud(n, 6, seed, lo=-3)
    ref = oc.build_kmap(c, 3, 1, dilate=True)
    km = sp.build_kmap(coords_dev(c), 3, 1, dilate=True)
    assert (km.n_in, km.n_out) == (ref.n_in, ref.n_out) and km.n_out > km.n_in
    np.testing.assert_array_equal(km.out_coords().cpu().numpy(), ref.out_coords)
    np.testing.assert_array_equal(km.in_coords().cpu().numpy(), c)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32), oc.bitmask(ref.M))
    assert km.n_pairs() == int((ref.M >= 0).sum()) == 27 * ref.n_in      # every input is read by 27 outputs
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, 32, 64, 27, "f16", seed)
    for n_split, kernel in ((0, 0), (1, 1), (2, 2)):
        cfg = sp.Config()
        cfg.n_split, cfg.kernel = n_split, kernel
        assert norm_err(sp.fwd(x, w, km, cfg), oc.forward(x32, w32, ref.M)) <= TOL["f16"]
        assert norm_err(sp.dgrad(g, w, km, cfg), oc.dgrad(g32, w32, ref.M, ref.n_in)) <= TOL["f16"]
    assert norm_err(sp.wgrad(x, g, km), oc.wgrad(x32, g32, ref.M)) <= 1e-4
    pw = km.pointwise(on_outputs=True)                                   # 1x1x1 layer over the dilated rows
    np.testing.assert_array_equal(pw.out_coords().cpu().numpy(), ref.out_coords)
    with pytest.raises(sp.SpconvError) as e:
        km.transpose()
    assert e.value.status == -1


def test_dilated_errors_and_k1(sp):
    import torch
    c = gen.uniform_cloud(200, 9, 53)
    ref = oc.build_kmap(c, 1, 1, dilate=True)                            # K = 1: the inputs, sorted
    km = sp.build_kmap(coords_dev(c), 1, 1, dilate=True)
    np.testing.assert_array_equal(km.out_coords().cpu().numpy(), ref.out_coords)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    edge = c.copy()
    edge[3] = (0, -32768, 5, 5)                                          # its neighbour at x - 1 cannot be packed
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(edge), 3, 1, dilate=True)
    assert e.value.status == -2
    dup = c.copy()
    dup[7] = dup[9]
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(dup), 3, 1, dilate=True)
    assert e.value.status == -3
    lib = sp.load_library()
    import ctypes
    out = ctypes.c_void_p()
    assert lib.spconv_build_kmap_dilated(None, 0, 5, None, ctypes.byref(out)) == -1
    assert lib.spconv_build_kmap_dilated(None, 0, 2, None, ctypes.byref(out)) == -1
    empty = sp.build_kmap(torch.empty((0, 4), dtype=torch.int32, device="cuda"), 3, 1, dilate=True)
    assert empty.n_out == 0


def _mask_words(big, words):
    """Python-int bitmasks -> uint32 [n][words], bit k in bit k % 32 of word k // 32."""
    out = np.zeros((len(big), words), np.uint32)
    for r, m in enumerate(big):
        m = int(m)
        for w in range(words):
            out[r, w] = (m >> (32 * w)) & 0xFFFFFFFF
    return out


@pytest.mark.parametrize("n,grid,lo", [(2000, 20, 0), (3000, 16, -8), (300, 7, 32760)])
def test_k5_submanifold_map_and_masks(sp, n, grid, lo):
    """K = 5 (125 offsets, Section 2.1's neighbourhood for any odd K): the library holds the map as five
    25-offset planes; what it exports is the whole map, bit for bit the oracle's, with 125-bit masks."""
    c = gen.uniform_cloud(n, grid, seed=500 + n, lo=lo)
    c[: n // 4, 0] = 3
    ref = oc.build_kmap(c, 5, 1)
    km = sp.build_kmap(coords_dev(c), 5, 1)
    assert (km.n_in, km.n_out, km.V) == (ref.n_in, ref.n_out, 125)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.in_coords().cpu().numpy(), ref.in_coords)
    np.testing.assert_array_equal(km.out_coords().cpu().numpy(), ref.out_coords)
    words = km.export_mask().cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(words, _mask_words(oc.bitmask(ref.M), 4))
    assert km.n_pairs() == int((ref.M >= 0).sum())
    km.destroy()


def test_k5_refusals(sp):
    """K = 5 exists as a submanifold map only; duplicates and rows beside the range fail as for K = 3."""
    c = gen.uniform_cloud(500, 16, seed=77)
    for stride, transposed in ((2, False), (1, True)):
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(c), 5, stride, transposed)
        assert e.value.status == -1
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(c), 5, 1, asynchronous=True)
    assert e.value.status == -1
    dup = np.concatenate([c, c[:1]])
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(dup), 5, 1)
    assert e.value.status == -3
    far = c.copy()
    far[3, 2] = 40000
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(far), 5, 1)
    assert e.value.status == -2
    km = sp.build_kmap(coords_dev(c), 5, 1)
    with pytest.raises(sp.SpconvError) as e:
        km.transpose()
    assert e.value.status == -1
    km.destroy()


@pytest.mark.parametrize("n,grid,lo", [(1, 1, 0), (12, 3, -32768), (13, 3, 32765), (49, 4, -3), (2401, 14, -32768)])
def test_k5_map_at_the_edges(sp, n, grid, lo):
    """Row counts around the probe's twelve rows per wave, runs of four cells cut by either end of the range."""
    c = gen.uniform_cloud(n, grid, seed=900 + n, lo=lo)
    ref = oc.build_kmap(c, 5, 1)
    km = sp.build_kmap(coords_dev(c), 5, 1)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32), _mask_words(oc.bitmask(ref.M), 4))
    assert km.n_pairs() == int((ref.M >= 0).sum())


@pytest.mark.parametrize("K,n_coarse", [(2, 1), (2, 9), (2, 1025), (3, 1), (3, 3), (3, 1025), (3, 65535), (3, 65545)])
def test_stride2_masks_by_rows_of_a_wave(sp, K, n_coarse):
    """Masks that are derived from finished map rows: whole and broken waves, on both sides of the 65,536 rows from
    which a wave of a 3x3x3 map takes 16 rows instead of two."""
    c = np.zeros((2 * n_coarse - 1, 4), np.int32)
    i = np.arange(2 * n_coarse - 1)
    c[:, 1], c[:, 3] = 4 * (i // 4000), i % 4000  # lines: their coarse points are n_coarse
    ref = _check_kmap(sp, c, K, 2, False)
    km = sp.build_kmap(coords_dev(c), K, 2)
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, 16, 16, K ** 3, "f16", n_coarse)
    assert norm_err(sp.dgrad(g, w, km), oc.dgrad(g32, w32, ref.M, ref.n_in)) <= 2e-2  # (walks the input side and its masks)


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("n,span,lo", [
    (1, (1, 1, 1), 0), (3, (2, 1, 3), -5), (64, (1, 1, 64), -1), (65, (1, 1, 130), 7), (900, (40, 1, 33), -21),
    (5000, (256, 64, 8), 1),           # one group of 16 words to a chunk
    (5000, (258, 66, 10), -3),         # two to some
    (26_000, (64, 64, 8), 3),          # groups of four words, hundreds of rows each
    (30_000, (700, 900, 500), -9),     # chunks of more words than LDS holds: two windows,
    (80_000, (1016, 1010, 1160), 0),   # three,
    (25_600, (800, 800, 652), 0),      # four
    (40, (60_000, 60_000, 60_000), -30_000), (2000, (1, 65_000, 64_000), -32_768),  # boxes that are left to the table: one
    (16_383, (3000, 3000, 3000), -7), (16_385, (3000, 3000, 3000), 9),              # or many workgroups, the verdict taken late or early,
    (100_000, (4000, 5000, 700), -2000), (150_000, (9000, 9000, 500), 1),           # keys of more than 32 bits
    (150_000, (1600, 1600, 1600), 0),  # K = 3: the sort of one launch per digit,
    (450_000, (2000, 2000, 2000), 0)])  # and the general one (from 393,217 coarse points on)
def test_stride2_boxes(sp, K, n, span, lo):
    """Stride-2 builds keep one bit per cell of the coarse points' box: boxes around word, chunk and workgroup limits, flat
    and long ones, negative and odd corners, several batches, and boxes too large for it, whose coarse points go through a hash table
    and a sort."""
    rng = np.random.default_rng(n + K)
    corners = np.array([[0] * 3, [s - 1 for s in span]])[:min(n, 2)]
    c = np.concatenate([corners, rng.integers(0, span, size=(2 * n, 3))])
    c = np.unique(np.concatenate([rng.integers(0, 3 if n < 1000 else 1, size=(len(c), 1)) * 2, c + lo], 1), axis=0)
    c = c[rng.permutation(len(c))][:n].astype(np.int32)
    _check_kmap(sp, c, K, 2, False)
    dup = np.concatenate([c, c[:1]])
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(dup), K, 2)
    assert e.value.status == -3


def test_stride2_box_and_table_too_large(sp):
    """Two million scattered rows: neither the bits of their box nor two hash tables in the bits' place are possible."""
    n = 2_200_000
    rng = np.random.default_rng(5)
    flat = np.unique(rng.integers(0, 60_000 ** 3, size=n))
    flat = flat[rng.permutation(len(flat))]
    p = np.stack([flat // 60_000 ** 2, flat // 60_000 % 60_000, flat % 60_000], 1) - 30_000
    c = np.concatenate([np.zeros((len(p), 1)), p], 1).astype(np.int32)
    km = sp.build_kmap(coords_dev(c), 2, 2)
    q = p // 2 + 40_000
    key, place = np.unique((q[:, 0] * 100_000 + q[:, 1]) * 100_000 + q[:, 2], return_inverse=True)
    want = np.stack([key // 100_000 ** 2, key // 100_000 % 100_000, key % 100_000], 1) - 40_000
    np.testing.assert_array_equal(km.out_coords().cpu().numpy()[:, 1:], want)
    M = np.full((len(key), 8), -1)
    d = p & 1
    M[place, d[:, 0] * 4 + d[:, 1] * 2 + d[:, 2]] = np.arange(len(p))
    np.testing.assert_array_equal(km.export().cpu().numpy(), M)
    km.destroy()


@pytest.mark.parametrize("K,n", [(3, 79_999), (3, 80_000), (3, 80_321), (5, 49_999), (5, 50_007)])
def test_submanifold_builds_on_both_sides_of_the_filter(sp, K, n):
    """5x5x5: from 50,000 rows on the probe keeps a filter of the existing runs (3x3x3 builds of these sizes go through buckets): half of the rows in a dense slab,
    half scattered, two batches, negative coordinates; and duplicates are still found."""
    rng = np.random.default_rng(n)
    c = np.concatenate([rng.integers(0, (300, 300, 3), size=(n, 3)), rng.integers(-9000, 9000, size=(n, 3))])
    c = np.unique(np.concatenate([rng.integers(0, 2, size=(2 * n, 1)), c], 1), axis=0)
    c = c[rng.permutation(len(c))][:n].astype(np.int32)
    _check_kmap(sp, c, K, 1, False) if K == 3 else _check_k5(sp, c)
    dup = np.concatenate([c[:-1], c[5:6]])
    with pytest.raises(sp.SpconvError) as e:
        sp.build_kmap(coords_dev(dup), K, 1)
    assert e.value.status == -3


def _check_k5(sp, c):
    ref = oc.build_kmap(c, 5, 1)
    km = sp.build_kmap(coords_dev(c), 5, 1)
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    assert km.n_pairs() == int((ref.M >= 0).sum())
    words = km.export_mask().cpu().numpy().view(np.uint32).reshape(-1, 4)
    present = ref.M >= 0
    for k in range(125):
        np.testing.assert_array_equal((words[:, k // 32] >> (k % 32)) & 1, present[:, k])


@pytest.mark.parametrize("n", [1, 2, 31, 1023, 1025, 2048, 2049, 4095, 5119, 5120, 5121, 9001])
@pytest.mark.parametrize("asynchronous", [False, True])
def test_small_submanifold_builds(sp, n, asynchronous):
    """Up to 5,120 rows a submanifold map is built in one launch: dense and scattered rows, corners of the coordinate range,
    and, waited for or not, duplicate rows and rows beside the range."""
    rng = np.random.default_rng(n)
    c = np.concatenate([rng.integers(0, (40, 40, 9), size=(n, 3)), rng.integers(-32768, 32768, size=(n, 3)),
                        [[-32768] * 3, [-32768, -32768, -32767], [32767] * 3, [32767, 32766, 32767]]])
    c = np.unique(np.concatenate([rng.integers(0, 2, size=(len(c), 1)) * 65534, c], 1), axis=0)
    c = c[rng.permutation(len(c))][:n].astype(np.int32)
    ref = oc.build_kmap(c, 3, 1)
    km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=asynchronous)
    if asynchronous:
        km.status()
    np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
    np.testing.assert_array_equal(km.in_coords().cpu().numpy(), ref.in_coords)
    np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32), oc.bitmask(ref.M))
    assert km.n_pairs() == int((ref.M >= 0).sum())
    for row, status in ((c[0], -3), ([0, 0, 40_000, 0], -2)):
        bad = np.concatenate([c, [row]]).astype(np.int32)
        with pytest.raises(sp.SpconvError) as e:
            km = sp.build_kmap(coords_dev(bad), 3, 1, asynchronous=asynchronous)
            if asynchronous:
                km.status()
        assert e.value.status == status


def test_unwaited_and_waited_builds_share_no_result(sp):
    """Two threads, each with its own stream and kmaps: one polls small asynchronous builds, the other waits for stride-2 builds.
    The pinned blocks that their figures arrive in go back and forth between them, each only after its last store."""
    import threading
    import torch
    small, big = gen.lidar_scene(12, target_n=700), gen.lidar_scene(13, target_n=2500)
    small_pairs = int((oc.build_kmap(small, 3, 1).M >= 0).sum())
    ref = oc.build_kmap(big, 3, 2)
    want = (ref.n_out, int((ref.M >= 0).sum()))
    small, big = coords_dev(small), coords_dev(big)
    torch.cuda.synchronize()
    wrong, start = [], threading.Barrier(2)

    def unwaited(stream):
        start.wait()
        for i in range(600):
            km = sp.build_kmap(small, 3, 1, stream=stream, asynchronous=True)
            if i % 3:
                km.status(stream)
            if i % 3 == 1 and km.n_pairs() != small_pairs:
                wrong.append(("small", km.n_pairs()))
            km.destroy()   # (unresolved every third time: the kmap's end waits for the block itself)

    def waited(stream):
        start.wait()
        for _ in range(400):
            km = sp.build_kmap(big, 3, 2, stream=stream)
            if (km.n_out, km.n_pairs()) != want:
                wrong.append(("big", km.n_out, km.n_pairs()))
            km.destroy()

    def run(f):
        try:
            f(torch.cuda.Stream())
        except Exception as e:  # (shown by the assertion below)
            wrong.append(repr(e))
    threads = [threading.Thread(target=run, args=(f,)) for f in (unwaited, waited)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not wrong, wrong[:5]


class _CountingAllocator:
    """Device memory for the library, counted; requests beyond `limit` live bytes are refused."""

    def __init__(self, sp, limit=None):
        self.sp, self.limit, self.live, self.most, self.refused = sp, limit, {}, 0, []

    def held(self):
        return sum(t.numel() for t in self.live.values())

    def __enter__(self):
        import gc
        import torch

        def alloc(n, stream):
            if self.limit is not None and self.held() + n > self.limit:
                self.refused.append(n)
                return 0
            t = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
            self.live[t.data_ptr()] = t
            self.most = max(self.most, self.held())
            return t.data_ptr()
        gc.collect()
        self.sp.set_allocator(alloc, lambda ptr, stream: self.live.pop(ptr))
        return self

    def __exit__(self, *_):
        import gc
        import torch
        gc.collect()
        torch.cuda.synchronize()
        self.sp.set_allocator(None, None)


@pytest.mark.parametrize("K,grid", [(2, 76), (3, 58)])
def test_stride2_kmaps_keep_what_their_outputs_need(sp, K, grid):
    """A dense cloud has an eighth as many outputs as inputs: the kmap does not stay as large as for one output per input, and
    works from the smaller tables."""
    from _util import TOL
    c = gen.full_grid(grid, 1, seed=3)
    ref = oc.build_kmap(c, K, 2)
    coords = coords_dev(c)
    with _CountingAllocator(sp) as mem:
        km = sp.build_kmap(coords, K, 2)
        V, rows_pad = K ** 3, -(-ref.n_out // 256) * 256
        tables = rows_pad * (V + 1) * 4 + ref.n_out * 16
        assert mem.held() <= len(c) * 16 + 2 * tables
        np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
        np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32), oc.bitmask(ref.M))
        np.testing.assert_array_equal(km.out_coords().cpu().numpy(), ref.out_coords)
        (x32, x), (w32, w), _ = make_layer(ref.n_in, ref.n_out, 16, 16, V, "f16", 4)
        assert norm_err(sp.fwd(x, w, km), oc.forward(x32, w32, ref.M)) <= TOL["f16"]
        km.destroy()
        assert not mem.live


@pytest.mark.parametrize("K", [2, 3])
def test_stride2_builds_where_memory_is_short(sp, K):
    """Where there is no room for tables of one output per input, a build that needs far less of them still succeeds."""
    c = gen.full_grid(30, 1, seed=4)
    ref = oc.build_kmap(c, K, 2)
    coords = coords_dev(c)
    _check_kmap(sp, c, K, 2, False)
    # room for the (fewer) bits and prefixes of a build over the box, cells and two sets of coordinates, but not for its map
    with _CountingAllocator(sp, limit=len(c) * (342 + 8 + 32) + 300_000) as mem:
        km = sp.build_kmap(coords, K, 2)
        assert -(-len(c) // 256) * 256 * K ** 3 * 4 in mem.refused
        np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
        km.destroy()
        assert not mem.live


@pytest.mark.parametrize("K", [2, 3])
def test_stride2_builds_over_fewer_cells_where_memory_is_short(sp, K):
    """Without 512 bytes a row for bits and prefixes, but with 384 of them: the box is still taken, and one that is too large for these is
    left to the table."""
    c = gen.lidar_scene(41, target_n=30_000)
    ref, n = oc.build_kmap(c, K, 2), len(c)
    far = _with_far_point(c, 1, 1900)
    for rows, over_box in ((c, True), (far, False)):
        with _CountingAllocator(sp, limit=n * (384 + 32 + 8 + 4 * K ** 3 + 4)) as mem:
            km = sp.build_kmap(coords_dev(rows), K, 2)
            assert mem.refused and mem.refused[0] >= 512 * n and mem.most > n * 350
            M = km.export().cpu().numpy()
            km.destroy()
            assert not mem.live
        np.testing.assert_array_equal(M, ref.M if over_box else oc.build_kmap(rows, K, 2).M)


@pytest.mark.parametrize("side,lo,batches", [(18, -32768, 1), (40, 32768 - 40, 1), (18, -9, 7), (12, 32768 - 12, 31)])
def test_dense_submanifold_builds_in_buckets(sp, side, lo, batches):
    """Blocks of 512 rows, several to a bucket: more rows than a workgroup looks up, and holds in its table, at a time; rows at both ends
    of the range; the same cells in several batches.  A row twice and a row beside the range fail such a build."""
    g = np.arange(lo, lo + side)
    c = np.stack(np.meshgrid(np.arange(batches), g, g, g, indexing="ij"), -1).reshape(-1, 4).astype(np.int32)
    c = c[np.random.default_rng(side).permutation(len(c))]
    _check_kmap(sp, c, 3, 1, False)
    km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=True)
    km.status()
    assert km.n_pairs() == int((oc.build_kmap(c, 3, 1).M >= 0).sum())
    for bad, status in ((np.vstack([c, c[len(c) // 2:][:1]]), -3), (np.vstack([c[:-1], [[0, 0, 40000, 0]]]).astype(np.int32), -2)):
        with pytest.raises(sp.SpconvError) as e:
            sp.build_kmap(coords_dev(bad), 3, 1)
        assert e.value.status == status


@pytest.mark.parametrize("n", [8191, 8193, 32769, 131071, 131329])
def test_scattered_submanifold_builds_in_buckets(sp, n):
    """On both sides of the numbers of buckets and of dealers; most blocks hold one row."""
    c = gen.uniform_cloud(n, 200, seed=n, lo=-100)
    c[: n // 3, 0] = 65534
    _check_kmap(sp, c, 3, 1, False)


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("n,side", [(1, 3), (63, 9), (64, 200), (257, 40), (1000, 11), (4099, 60)])
def test_input_side_of_stride2_maps(sp, K, n, side):
    """Made from the rows' candidates, and searched where these would be more than the output side is (3x3x3, 1,000 rows): around the
    ends of waves and of the padding, coordinates of both signs."""
    rng = np.random.default_rng(n)
    flat = rng.permutation(side ** 3)[:n]
    c = np.stack([rng.integers(0, 1 if 2 * n > side ** 3 else 2, n), *np.unravel_index(flat, (side,) * 3)], 1).astype(np.int32)
    c[:, 1:] -= side // 2
    ref = oc.build_kmap(c, K, 2)
    up = sp.build_kmap(coords_dev(c), K, 2).transpose()
    T = np.full((n, K ** 3), -1, np.int32)
    out, k = np.nonzero(ref.M >= 0)
    T[ref.M[out, k], k] = out
    np.testing.assert_array_equal(up.export().cpu().numpy(), T)
    np.testing.assert_array_equal(up.export_mask().cpu().numpy().view(np.uint32), oc.bitmask(T))


@pytest.mark.parametrize("n,cells,side", [(6000, 1, 1), (300_000, 1, 1), (300_000, 3, 12), (300_000, 1700, 12), (60_000, 30_000, 32)])
def test_submanifold_builds_over_rows_that_share_cells(sp, n, cells, side):
    """Any number of rows in one cell (rows padded with zeros), in a few, or in all cells of many blocks: the build fails, in a time
    that grows with the rows (a walk of the one bucket to its end takes 115,000 passes with 300,000 of them, tenths of a second, against
    30 ms asked for here), and what an unwaited one leaves in its map are rows or nothing, which a layer may walk before the status is
    asked for."""
    import time
    import torch
    rng = np.random.default_rng(n + cells)
    at = np.stack(np.unravel_index(np.arange(cells), (side,) * 3), 1)
    dup = np.concatenate([np.zeros((n, 1)), at[rng.integers(0, cells, n)]], 1).astype(np.int32)
    cloud = gen.uniform_cloud(4000, 60, seed=n, lo=20)
    for c in (dup, rng.permutation(np.concatenate([cloud, dup]))):
        coords = coords_dev(c)
        torch.cuda.synchronize()
        took = []
        for _ in range(3):
            t0 = time.perf_counter()
            with pytest.raises(sp.SpconvError) as e:
                sp.build_kmap(coords, 3, 1)
            took.append(time.perf_counter() - t0)
            assert e.value.status == -3
        assert min(took) < 0.03, took
        km = sp.build_kmap(coords, 3, 1, asynchronous=True)
        x, w = torch.ones(len(c), 16, dtype=torch.float16, device="cuda"), torch.ones(27, 16, 16, dtype=torch.float16, device="cuda")
        assert torch.isfinite(sp.fwd(x, w, km, sp.Config(n_split=0, kernel=1))).all()
        M = km.export().cpu().numpy()
        assert M.min() >= -1 and M.max() < len(c)
        with pytest.raises(sp.SpconvError) as e:
            km.status()
        assert e.value.status == -3
        km.destroy()


def _with_far_point(c, axis, cells_per_row):
    """c and one more point, as far along an axis as makes the box of the coarse points that many cells a row (or as far as can be)."""
    q = c.astype(np.int64) >> np.array([0, 1, 1, 1])
    span = q.max(0) - q.min(0) + 1
    p = c[:1].copy()
    p[0, axis] = min(c[:, axis].min() + 2 * (int(cells_per_row * len(c)) * int(span[axis]) // int(np.prod(span))), 32_767)
    return np.concatenate([c, p])


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("shape", ["plane", "wall", "block"])
def test_stride2_boxes_with_rows_in_a_small_part(sp, K, shape):
    """Rows that crowd into a part of the box: a plane or a block with one point far from it (more rows to a window than are taken one by
    one), a wall whose cells stand at a regular distance (a multiple of a run of groups) from each other."""
    g = np.random.default_rng(K)
    if shape == "plane":
        c = np.stack(np.meshgrid([5], np.arange(-120, 120), np.arange(250), indexing="ij"), -1).reshape(-1, 3)
    elif shape == "wall":
        c = np.stack(np.meshgrid(np.arange(320), [3], np.arange(64), indexing="ij"), -1).reshape(-1, 3)
        c = np.concatenate([c, [[0, 0, 0], [319, 1023, 255]]])  # (512 cells by 128 to a step along x: 2048 words)
    else:
        c = np.stack(np.meshgrid(*[np.arange(-20, 20)] * 3, indexing="ij"), -1).reshape(-1, 3)
    c = np.concatenate([np.zeros((len(c), 1)), c], 1).astype(np.int32)[g.permutation(len(c))]
    for axis in (1, 2, 3) if shape != "wall" else (0,):
        _check_kmap(sp, _with_far_point(c, axis, 1500) if axis else c, K, 2, False)


def test_stride2_build_with_a_far_point_takes_little_longer(sp):
    """A plane of 200,000 rows and one point far from it: the plane's rows are shared among workgroups (in one of them, the build took 5.3
    times as long as without the point; 1.2 to 1.3 times as it is)."""
    import time
    import torch
    c = np.stack(np.meshgrid([0], [0], np.arange(400), np.arange(500), indexing="ij"), -1).reshape(-1, 4).astype(np.int32)
    c[:, 2:] += np.random.default_rng(1).integers(0, 2, size=(len(c), 2)) + c[:, 2:]  # (one row in each 2 x 2)
    c = np.random.default_rng(2).permutation(c)
    best = []
    for rows in (c, _with_far_point(c, 1, 1500)):
        coords, took = coords_dev(rows), []
        for _ in range(12):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sp.build_kmap(coords, 3, 2).destroy()
            torch.cuda.synchronize()
            took.append(time.perf_counter() - t0)
        best.append(min(took))
    assert best[1] < 2.5 * best[0], best


@pytest.mark.parametrize("K", [2, 3])
def test_candidates_go_when_the_input_side_is_there(sp, K):
    """What a stride-2 kmap holds beside its tables is given back: with the input side that is made from it, and when plans are dropped
    (behind which the input side is searched for, and the same)."""
    from _util import TOL
    c = gen.lidar_scene(31, target_n=20_000)
    ref = oc.build_kmap(c, K, 2)
    V, n = K ** 3, len(c)
    out_pad, in_pad = -(-ref.n_out // 256) * 256, -(-n // 256) * 256
    (x32, x), (w32, w), (g32, g) = make_layer(ref.n_in, ref.n_out, 16, 16, V, "f16", 4)
    want, coords, map_order = oc.dgrad(g32, w32, ref.M, ref.n_in), coords_dev(c), sp.Config(n_split=0)
    tables = n * 16 + max(ref.n_out, n) * 16 + max(out_pad, in_pad) * (V + 1) * 4  # (at most: made for as many outputs as inputs)
    with _CountingAllocator(sp) as mem:
        km = sp.build_kmap(coords, K, 2)
        built = mem.held()
        assert built > tables
        assert norm_err(sp.dgrad(g, w, km, map_order), want) <= TOL["f16"]
        km.n_pairs()
        assert mem.held() <= tables + in_pad * (V + 1) * 4
        for _ in range(2):
            km.drop_plans()
            assert mem.held() <= tables
            assert norm_err(sp.dgrad(g, w, km, map_order), want) <= TOL["f16"]
        km.destroy()
        km = sp.build_kmap(coords, K, 2)
        assert mem.held() == built
        km.drop_plans()
        assert mem.held() <= tables
        assert norm_err(sp.dgrad(g, w, km, map_order), want) <= TOL["f16"]
        km.destroy()
        assert not mem.live


@pytest.mark.parametrize("K", [2, 3])
def test_partner_of_a_kmap_that_goes_at_once(sp, K):
    """The partner's table is made on another stream, from what the source's build left; the source goes before that has run, and its
    memory to builds on its own stream."""
    import torch
    c = gen.lidar_scene(32, target_n=30_000)
    ref = oc.build_kmap(c, K, 2)
    T = np.full((len(c), K ** 3), -1, np.int32)
    out, k = np.nonzero(ref.M >= 0)
    T[ref.M[out, k], k] = out
    coords, other = coords_dev(c), coords_dev(c[::-1].copy())
    here, there = torch.cuda.Stream(), torch.cuda.Stream()
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    for _ in range(5):
        km = sp.build_kmap(coords, K, 2, stream=here)
        with torch.cuda.stream(there):
            for _ in range(4):
                busy @ busy   # (the partner's launch waits behind these)
        up = km.transpose(stream=there)
        km.destroy()
        for _ in range(3):
            sp.build_kmap(other, K, 2, stream=here).destroy()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(up.export().cpu().numpy(), T)
        up.destroy()


@pytest.mark.parametrize("asynchronous", [False, True])
def test_submanifold_builds_where_memory_is_short(sp, asynchronous):
    """Without room for the buckets (96 bytes a row and more) the map is built over a table, as it was where 64 were enough; failed builds
    report as ever, waited for or not, and what an unwaited one leaves can be walked."""
    c = gen.uniform_cloud(60_000, 80, seed=3, lo=-40)
    ref, n = oc.build_kmap(c, 3, 1), len(c)
    pad = -(-n // 256) * 256
    with _CountingAllocator(sp, limit=n * (16 + 75) + pad * 28 * 4 + 100_000) as mem:
        km = sp.build_kmap(coords_dev(c), 3, 1, asynchronous=asynchronous)
        assert mem.refused and min(mem.refused) >= 96 * n
        np.testing.assert_array_equal(km.export().cpu().numpy(), ref.M)
        np.testing.assert_array_equal(km.export_mask().cpu().numpy().view(np.uint32)[:n], oc.bitmask(ref.M))
        np.testing.assert_array_equal(km.in_coords().cpu().numpy(), c)
        km.status()
        assert km.n_pairs() == int((ref.M >= 0).sum())
        km.destroy()
        for row, status in ((c[5], -3), ([0, 0, 40_000, 0], -2)):
            bad = c.copy()
            bad[n // 2] = row
            if not asynchronous:
                with pytest.raises(sp.SpconvError) as e:
                    sp.build_kmap(coords_dev(bad), 3, 1)
            else:
                km = sp.build_kmap(coords_dev(bad), 3, 1, asynchronous=True)
                M = km.export().cpu().numpy()
                assert M.min() >= -1 and M.max() < n
                for _ in range(2):
                    with pytest.raises(sp.SpconvError) as e:
                        km.status()
                km.destroy()
            assert e.value.status == status
        assert not mem.live
