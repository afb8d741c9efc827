"""GPU parity, layer by layer (teacher-forced): every HIP layer is fed the oracle's inputs and
state for a frame and must reproduce the oracle's outputs and state -- masks, index lists and
all element-wise arithmetic bit-exactly, convolution sums within the stated tolerance.
All calls go through the C ABI (ctypes binding)."""
import numpy as np
import pytest
import torch

import paper_2203_03996_amd as pkg
from oracle import deltacnn_oracle as orc
from oracle.deltacnn_oracle import Delta as ODelta
from tests.helpers import NP_DTYPE, TOL, U32, check_delta, rel_err, sum_slack, to_np, ulp, upload_delta

pytestmark = pytest.mark.gpu
DT = {"f32": pkg.F32, "f16": pkg.F16}
TDT = {"f32": torch.float32, "f16": torch.float16}


def _rand_delta(rng, shape, density, S, scale=1.0):
    """Random delta whose unflagged pixels are NaN (reading them would poison the result)."""
    n, h, w, c = shape
    mask = (rng.random((n, h, w)) < density).astype(np.uint8)
    data = (rng.normal(0, scale, shape)).astype(NP_DTYPE[S])
    return ODelta(data, mask).poisoned()


def _upload(d: ODelta):
    return upload_delta(d.data, d.mask)


# ---- mask propagation + compaction (bit-exact) --------------------------------------------------
@pytest.mark.parametrize("n,h,w", [(1, 64, 64), (3, 37, 53), (2, 128, 128), (1, 7, 5)])
@pytest.mark.parametrize("k,stride,pad", [(1, 1, 0), (3, 1, 1), (3, 2, 1), (7, 2, 3), (1, 2, 0)])
@pytest.mark.parametrize("density", [0.0, 0.03, 0.5, 1.0])
def test_mask_compact(n, h, w, k, stride, pad, density):
    rng = np.random.default_rng(n * 1000 + h + k * 7 + int(density * 100))
    m = (rng.random((n, h, w)) < density).astype(np.uint8)
    ctx = pkg.Context(n * h * w)
    mo, idx, cnt = ctx.mask_compact(torch.from_numpy(m).cuda(), k, stride, pad)
    ctx.sync()
    ref = orc.window_mask(m, k, stride, pad)
    assert np.array_equal(to_np(mo), ref)
    ridx, rcnt = orc.compact(ref)
    assert int(to_np(cnt)[0]) == rcnt
    assert np.array_equal(to_np(idx)[:rcnt], ridx)


def test_mask_union():
    rng = np.random.default_rng(5)
    a = (rng.random((2, 33, 47)) < 0.1).astype(np.uint8)
    b = (rng.random((2, 33, 47)) < 0.1).astype(np.uint8)
    ctx = pkg.Context(a.size)
    mo, idx, cnt = ctx.mask_compact(torch.from_numpy(a).cuda(), 1, 1, 0, mask_b=torch.from_numpy(b).cuda())
    ctx.sync()
    assert np.array_equal(to_np(mo), a | b)
    assert np.array_equal(to_np(idx)[:int(to_np(cnt)[0])], np.flatnonzero((a | b).reshape(-1)))


# ---- input delta generation (bit-exact) ---------------------------------------------------------
@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("shape,r", [((1, 64, 64, 32), 0), ((2, 45, 31, 64), 0), ((1, 40, 56, 3), 0), ((1, 9, 9, 17), 0),
                                     ((1, 16, 16, 1024), 0),
                                     # input-mask dilation by the (2r+1)^2 square (Section 4)
                                     ((2, 45, 31, 64), 1), ((1, 64, 72, 16), 7), ((1, 9, 9, 17), 3), ((3, 20, 20, 8), 15)])
def test_deltagen(S, shape, r):
    rng = np.random.default_rng(sum(shape) + r)
    n, h, w, c = shape
    ref = orc.DeltaGen(0.3, r, S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.DELTAGEN, DT[S], n, h, w, c, eps=0.3, dilate_r=r))
    f0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    r0 = ref.init(f0)
    g0 = layer.init([torch.from_numpy(f0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), r0)
    frame = f0.astype(np.float64)
    for t in range(4):
        frame = frame + (rng.random((n, h, w, 1)) < (0.2 if r == 0 else 0.02)) * rng.normal(0, 0.4, shape)
        fr = frame.astype(NP_DTYPE[S])
        want = ref.step(fr).poisoned()
        out = layer.step([pkg.Delta(torch.from_numpy(fr).cuda(), None, None, None)])
        ctx.sync()
        check_delta(out, want, S, f"deltagen frame {t}", exact_values=True)
        assert np.array_equal(to_np(layer.state_tensor(0)), ref.P)
    st = layer.stats()
    assert st["pixels_out"] == want.count and st["pixels_total"] == n * h * w


# ---- activation + truncation (bit-exact) ---------------------------------------------------------
@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("f,carry", [("relu", False), ("relu6", False), ("relu", True)])
@pytest.mark.parametrize("shape", [(1, 64, 64, 32), (2, 33, 29, 64), (1, 24, 24, 256), (1, 12, 12, 960),
                                   (1, 10, 10, 2048), (1, 9, 11, 3), (1, 9, 11, 17), (1, 8, 8, 100),
                                   # wide pixels on short lists: the channels of a pixel are split over a workgroup's waves
                                   (2, 9, 7, 1024), (1, 5, 5, 1536), (3, 6, 7, 512)])
def test_act_trunc(S, f, carry, shape):
    """carry: the variant that leaves the rounding residue of x^A in x^T on an update (bit-exact like the rest)."""
    rng = np.random.default_rng(sum(shape) + len(f))
    n, h, w, c = shape
    eps = 0.35
    ref = orc.ActTrunc(f, eps, S, carry=carry)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, DT[S], n, h, w, c, act=pkg.ACT_CODES[f], eps=eps, xT_residue=int(carry)))
    x0 = rng.normal(0, 2, shape).astype(NP_DTYPE[S])
    r0 = ref.init(x0)
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), r0)
    assert np.array_equal(to_np(layer.state_tensor(0)), ref.xA)
    saw = set()
    for t in range(4):
        d = _rand_delta(rng, shape, [0.3, 0.05, 1.0, 0.0][t], S, scale=0.3)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"act frame {t}", exact_values=True)
        assert np.array_equal(to_np(layer.state_tensor(0)), ref.xA)
        assert np.array_equal(to_np(layer.state_tensor(1)), ref.xT)
        if want.count:
            saw.add("upd")
        if want.count < d.count:
            saw.add("trunc")
    assert "upd" in saw and ("trunc" in saw or c > 64)     # wide pixels always exceed the threshold
    if carry and S == "f16":
        assert np.any(ref.xT[want.mask == 1] != 0) if want.count else True


@pytest.mark.parametrize("shape", [(2, 40, 37, 64), (1, 9, 7, 1024)])
def test_layer_whose_list_nobody_walks_keeps_no_count_and_alternates_its_masks(shape):
    """want_idx = 0: the view hands out no count (nothing on a step's path keeps one) and dcnn_layer_stats counts
    the mask instead; the layer walks its input's list, so it alternates between two output masks, each cleared a
    step ahead -- frames whose lists are disjoint, full and empty in turn must leave no stale flag behind."""
    S, f, eps = "f16", "relu", 0.35
    rng = np.random.default_rng(shape[3])
    n, h, w, c = shape
    ref = orc.ActTrunc(f, eps, S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, DT[S], n, h, w, c, act=pkg.ACT_CODES[f], eps=eps, want_idx=0))
    x0 = rng.normal(0, 2, shape).astype(NP_DTYPE[S])
    ref.init(x0)
    layer.init([torch.from_numpy(x0).cuda()])
    masks = set()
    for t, dens in enumerate([0.4, 0.4, 1.0, 0.0, 0.1, 0.0, 0.6]):
        d = _rand_delta(rng, shape, dens, S, scale=0.3)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        assert out.count is None
        masks.add(out.mask.data_ptr())
        assert np.array_equal(to_np(out.mask), want.mask), f"frame {t}"
        assert layer.stats()["pixels_out"] == want.count and layer.stats()["pixels_in"] == d.count
        sel = want.mask.astype(bool)
        assert np.array_equal(to_np(out.data)[sel], want.data[sel])
    assert len(masks) == 2


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("act", ["relu", "none"])
@pytest.mark.parametrize("shape", [(2, 31, 30, 64), (2, 11, 9, 2048), (1, 13, 5, 1024)])
def test_add_act(S, act, shape):
    rng = np.random.default_rng(17)
    n, h, w, c = shape
    eps = 0.4
    radd, ract = orc.Add(S), orc.ActTrunc(act, eps, S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, DT[S], n, h, w, c, act=pkg.ACT_CODES[act], eps=eps, n_in=2))
    a0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    b0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    r0 = radd.init(a0, b0)
    if act != "none":
        r0 = ract.init(r0)
    g0 = layer.init([torch.from_numpy(a0).cuda(), torch.from_numpy(b0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), r0)
    for t in range(3):
        da = _rand_delta(rng, shape, 0.2, S, 0.3)
        db = _rand_delta(rng, shape, 0.1, S, 0.3)
        want = radd.step(da, db).poisoned()
        if act != "none":
            want = ract.step(want).poisoned()
        out = layer.step([_upload(da), _upload(db)])
        ctx.sync()
        check_delta(out, want, S, f"add+{act} frame {t}", exact_values=True)
        if act != "none":
            assert np.array_equal(to_np(layer.state_tensor(0)), ract.xA)
            assert np.array_equal(to_np(layer.state_tensor(1)), ract.xT)


@pytest.mark.parametrize("S,c", [("f16", 1024), ("f16", 2048), ("f32", 512), ("f32", 1024)])
@pytest.mark.parametrize("nhw", [(1, 1, 1), (1, 5, 13), (1, 7, 12), (2, 8, 8), (1, 11, 13), (4, 22, 22)])
def test_wide_add_act_builds_its_list_on_any_pixel_count(S, c, nhw):
    """The tile count is rounded up to whole tiles while the map ends inside one: 1, 65, 84, 128, 143 and 1936 pixels end 1, 1,
    20, 32, 15 and 16 entries into their last tile, listed in full, in part and not at all."""
    rng = np.random.default_rng(c + nhw[1])
    n, h, w = nhw
    shape, eps = (n, h, w, c), 0.4
    radd, ract = orc.Add(S), orc.ActTrunc("relu", eps, S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, DT[S], n, h, w, c, act=pkg.ACT_RELU, eps=eps, n_in=2, want_idx=0))
    dense = [rng.normal(0, 1, shape).astype(NP_DTYPE[S]) for _ in range(2)]
    ract.init(radd.init(*dense))
    layer.init([torch.from_numpy(a).cuda() for a in dense])
    for t, (d0, d1) in enumerate([(1.0, 1.0), (0.2, 0.1), (0.97, 0.5), (0.0, 0.0), (1.0, 0.0)]):
        da, db = _rand_delta(rng, shape, d0, S, 0.15), _rand_delta(rng, shape, d1, S, 0.15)
        want = ract.step(radd.step(da, db).poisoned()).poisoned()
        out = layer.step([_upload(da), _upload(db)])
        ctx.sync()
        check_delta(out, want, S, f"frame {t}", exact_values=True)
        assert np.array_equal(to_np(layer.state_tensor(0)), ract.xA), f"frame {t}"
        assert np.array_equal(to_np(layer.state_tensor(1)), ract.xT), f"frame {t}"


# ---- convolution: linear (values within tolerance; masks and lists bit-exact) -------------------
CONV_CASES = [
    # S, k, stride, pad, cin, cout, (n,h,w)
    ("f32", 3, 1, 1, 32, 32, (1, 64, 64)),
    ("f32", 1, 1, 0, 32, 64, (2, 20, 23)),
    ("f32", 3, 2, 1, 16, 48, (1, 31, 33)),
    ("f32", 3, 1, 1, 3, 32, (1, 30, 30)),
    ("f16", 1, 1, 0, 64, 64, (2, 40, 40)),
    ("f16", 3, 1, 1, 64, 64, (2, 40, 37)),
    ("f16", 1, 1, 0, 64, 256, (1, 48, 48)),
    ("f16", 3, 2, 1, 3, 32, (1, 50, 50)),
    ("f16", 7, 2, 3, 3, 64, (1, 40, 40)),
    # few input channels: the window's (tap, channel) pairs are one flat K dimension
    ("f16", 5, 1, 2, 6, 32, (1, 18, 20)),
    ("f32", 5, 2, 2, 3, 16, (2, 17, 19)),
    ("f16", 3, 1, 1, 1, 8, (1, 12, 16)),
    ("f16", 7, 1, 3, 5, 40, (1, 15, 15)),
    ("f16", 1, 1, 0, 48, 96, (1, 25, 25)),
    ("f16", 3, 1, 1, 32, 160, (1, 21, 20)),
    ("f16", 1, 2, 0, 64, 128, (1, 30, 30)),
    ("f16", 3, 1, 1, 64, 16, (1, 24, 24)),
    # weights too large for LDS: streamed in slices; the last two are wider than one staging tile
    ("f16", 3, 2, 1, 64, 128, (1, 30, 30)),
    ("f16", 3, 1, 1, 256, 256, (1, 20, 20)),
    ("f16", 1, 1, 0, 160, 960, (1, 14, 14)),
    ("f16", 1, 1, 0, 512, 2048, (1, 9, 8)),
    ("f32", 3, 1, 1, 128, 128, (1, 16, 16)),
    ("f32", 1, 1, 0, 64, 1024, (1, 12, 12)),
    # long work lists on streamed weights (sparse steps: several pixel tiles per wave share the weight operands):
    # two / four waves per tile, an input's own list, a strided window, fp32, and two passes over the channels
    ("f16", 3, 1, 1, 128, 128, (6, 128, 128)),
    ("f16", 1, 1, 0, 256, 512, (4, 96, 96)),
    ("f16", 3, 2, 1, 128, 256, (8, 128, 128)),
    ("f32", 3, 1, 1, 64, 128, (6, 96, 96)),
    ("f16", 1, 1, 0, 256, 1024, (4, 80, 80)),
]


def _near_tie(ract, eps, slack):
    """Pixels whose decision the arithmetic leaves open: the oracle's max-norm lies within the value
    tolerance of the threshold, or within what the pixel's own intermediates may differ by."""
    u = np.nan_to_num(ract.last_u, nan=np.inf)
    return np.abs(u - eps) <= TOL[ract.S] * abs(eps) + np.asarray(slack).max(axis=-1)


def _conv_layers(S, k, stride, pad, cin, cout, nhw, rng, act=pkg.ACT_NONE, eps=0.0, n_in=1, depthwise=False):
    n, h, w = nhw
    if depthwise:
        wgt = (rng.normal(0, 1, (k, k, cin)) * np.sqrt(2.0 / (k * k))).astype(NP_DTYPE[S])
    else:
        wgt = (rng.normal(0, 1, (k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(NP_DTYPE[S])
    bias = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
    ref = orc.Conv(wgt, bias, stride, pad, depthwise, S)
    ctx = pkg.Context(n * h * w)
    desc = pkg.make_desc(pkg.DWCONV if depthwise else pkg.CONV, DT[S], n, h, w, cin, k=k, stride=stride, pad=pad,
                         cout=cout, act=act, eps=eps, n_in=n_in)
    layer = pkg.Layer(ctx, desc, torch.from_numpy(wgt).cuda(), torch.from_numpy(bias).cuda())
    return ctx, layer, ref


@pytest.mark.parametrize("S,k,stride,pad,cin,cout,nhw", CONV_CASES)
def test_conv_linear(S, k, stride, pad, cin, cout, nhw):
    rng = np.random.default_rng(k * 100 + cin + cout)
    n, h, w = nhw
    ctx, layer, ref = _conv_layers(S, k, stride, pad, cin, cout, nhw, rng)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    r0 = ref.init(x0)
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert rel_err(to_np(g0), r0, slack=sum_slack(ref, x0, bias=True)) <= TOL[S], "dense first frame"
    for t, dens in enumerate([0.05, 0.4, 1.0, 0.0]):
        d = _rand_delta(rng, (n, h, w, cin), dens, S)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"conv frame {t} density {dens}", slack=sum_slack(ref, d.zero_filled()))
        st = layer.stats()
        assert st["pixels_in"] == d.count and st["pixels_out"] == want.count


@pytest.mark.parametrize("pattern", ["columns3", "rows3", "diagonal", "holes", "border"])
@pytest.mark.parametrize("nhw", [(2, 40, 37), (1, 33, 64)])
def test_conv3x3_row_gathers_on_structured_masks(pattern, nhw):
    """3x3 / stride 1 / padding 1 on a resident-weight layer with masks that list (nearly) the whole map while
    every pixel has only some taps flagged: the kernel then fetches one centre column per window row and takes the
    left / right taps from neighbouring lanes -- across tile boundaries, row ends and images."""
    S, cin, cout = "f16", 64, 64
    rng = np.random.default_rng(len(pattern) * 7 + nhw[1])
    n, h, w = nhw
    ctx, layer, ref = _conv_layers(S, 3, 1, 1, cin, cout, nhw, rng)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    ref.init(x0)
    layer.init([torch.from_numpy(x0).cuda()])
    yy, xx = np.meshgrid(np.arange(h), np.arange(w), indexing="ij")
    mask2d = {"columns3": xx % 3 == 0, "rows3": yy % 3 == 1, "diagonal": (xx + yy) % 3 == 0,
              "holes": (xx * 7 + yy * 13) % 11 != 0, "border": (xx == 0) | (xx == w - 1) | (yy % 2 == 0)}[pattern]
    mask = np.broadcast_to(mask2d, (n, h, w)).astype(np.uint8).copy()
    mask[-1, h // 2:, : w // 3] = 0                      # a corner of the last image without any flag
    data = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    d = ODelta(data, mask).poisoned()
    want = ref.step(d).poisoned()
    out = layer.step([_off_alignment(_upload(d))])       # (a list from memory: blocks compacted in place are gathered tap by tap)
    ctx.sync()
    assert want.count * 4 >= n * h * w * 3, "the pattern must list at least three quarters of the map"
    check_delta(out, want, S, f"row gathers, {pattern}", slack=sum_slack(ref, d.zero_filled()))


@pytest.mark.parametrize("S,cin,cout", [("f16", 64, 64), ("f16", 136, 24), ("f16", 24, 64), ("f32", 20, 40)] + [
    # weights too large for LDS, tiles of one, two and four waves with one to four column blocks, whole and broken lines of channels
    ("f16", 136, 64), ("f16", 128, 96), ("f16", 128, 128), ("f16", 104, 192), ("f16", 72, 256), ("f16", 64, 384), ("f16", 264, 32), ("f32", 72, 64)])
def test_conv3x3_of_a_stream_has_the_same_bits_alone_and_in_a_batch(S, cin, cout):
    """One stream of 7 K pixels compacts blocks in place and gathers tap by tap; ten of them take a list from memory and, with most
    of the map listed and weights resident in LDS, one gather per window row.  One to five groups of K-steps, the last one whole or not."""
    rng = np.random.default_rng(cin)
    n, h, w = 10, 89, 83
    dt = NP_DTYPE[S]
    wgt = torch.from_numpy((rng.standard_normal((3, 3, cin, cout)) * np.sqrt(2.0 / (9 * cin))).astype(dt)).cuda()
    layers = []
    for streams in (1, n):
        ctx = pkg.Context(streams * h * w)
        desc = pkg.make_desc(pkg.CONV, DT[S], streams, h, w, cin, k=3, stride=1, pad=1, cout=cout, act=pkg.ACT_RELU, eps=0.3, want_idx=0)
        layers.append((ctx, pkg.Layer(ctx, desc, wgt)))
    first = torch.from_numpy(rng.standard_normal((n, h, w, cin)).astype(dt)).cuda()
    for (ctx, layer), frame in zip(layers, (first[3:4].contiguous(), first)):
        layer.init([frame])
    for dens in (1.0, 0.5, 0.03, 0.95):
        d = _rand_delta(rng, (n, h, w, cin), dens, S, 0.4)
        alone = layers[0][1].step([_upload(ODelta(d.data[3:4].copy(), d.mask[3:4].copy()))])
        batch = layers[1][1].step([_upload(d)])
        for ctx, _ in layers:
            ctx.sync()
        mask = to_np(alone.mask)[0]
        assert np.array_equal(to_np(batch.mask)[3], mask), f"density {dens}: mask"
        assert np.array_equal(to_np(batch.data)[3][mask == 1], to_np(alone.data)[0][mask == 1]), f"density {dens}: values"


@pytest.mark.parametrize("pattern", ["all", "holes", "sevenths"])
@pytest.mark.parametrize("S,cin,cout", [("f16", 128, 128), ("f32", 64, 128)])
def test_conv3x3_row_gathers_on_the_register_blocked_kernel(S, cin, cout, pattern):
    """The same window-row gathers on a layer whose weights do not fit LDS, with a list long enough for several
    pixel tiles per wave (more than 65,536 entries) and at least three quarters of all window taps flagged.  fp32: three
    tiles per wave, left / right taps from neighbouring lanes, the tiles' edge columns fetched separately.  fp16, whose
    waves share their gathers through LDS: the same lists tap by tap."""
    nhw = (5, 128, 136)
    rng = np.random.default_rng(len(pattern) * 11 + cin)
    n, h, w = nhw
    ctx, layer, ref = _conv_layers(S, 3, 1, 1, cin, cout, nhw, rng)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    ref.init(x0)
    layer.init([torch.from_numpy(x0).cuda()])
    yy, xx = np.meshgrid(np.arange(h), np.arange(w), indexing="ij")
    mask2d = {"all": xx >= 0, "holes": (xx * 7 + yy * 13) % 11 != 0, "sevenths": (xx * 5 + yy * 3) % 7 != 0}[pattern]
    mask = np.broadcast_to(mask2d, (n, h, w)).astype(np.uint8).copy()
    mask[-1, h - 9:, : w // 3] = 0                       # a corner of the last image without any flag
    data = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    d = ODelta(data, mask).poisoned()
    want = ref.step(d).poisoned()
    out = layer.step([_upload(d)])
    ctx.sync()
    assert want.count > 65536 and d.count * 4 >= want.count * 3, "long list, at least three quarters of the taps flagged"
    check_delta(out, want, S, f"row gathers, register-blocked, {pattern}", slack=sum_slack(ref, d.zero_filled()))


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,res", [
    # streamed weights, long lists, fused tail: two waves per tile with a residual, four waves per tile, three
    # column blocks per wave in fp32
    ("f16", 3, 1, 128, 128, (5, 128, 136), True),
    ("f16", 1, 1, 256, 256, (4, 96, 96), True),
    ("f32", 3, 1, 64, 96, (6, 96, 96), True),
    ("f32", 3, 1, 32, 32, (1, 64, 64), False),
    ("f16", 1, 1, 64, 64, (2, 32, 32), False),
    ("f16", 3, 1, 64, 64, (2, 33, 35), False),
    ("f16", 1, 1, 64, 256, (1, 40, 40), True),
    ("f16", 3, 2, 64, 128, (1, 30, 30), False),
    ("f16", 3, 2, 3, 32, (1, 40, 40), False),
    ("f32", 1, 1, 16, 16, (1, 20, 20), True),
    # further shapes of the wave-specialised kernel: strided resident 3x3, channels that do not fill the
    # last K-step, three column blocks per wave, two and four waves per tile with a residual, fp32 wide
    ("f16", 3, 2, 32, 32, (2, 41, 37), False),
    ("f16", 1, 1, 24, 96, (1, 33, 31), False),
    ("f16", 3, 1, 16, 96, (1, 31, 29), True),
    ("f16", 1, 1, 64, 128, (1, 45, 40), True),
    ("f16", 1, 2, 32, 256, (1, 50, 44), True),
    ("f32", 1, 1, 32, 64, (1, 37, 30), True),
    ("f32", 3, 1, 16, 64, (3, 21, 22), False),
    ("f16", 1, 1, 64, 64, (4, 96, 96), False),
    # output channels that do not fill the last column block (padded lanes must stay out of the maximum)
    ("f16", 1, 1, 32, 72, (1, 29, 33), True),
    ("f16", 3, 1, 32, 40, (1, 23, 27), False),
    ("f32", 1, 1, 16, 44, (1, 23, 27), False),
])
def test_conv_fused_act(S, k, stride, cin, cout, nhw, res):
    """conv (+ residual) + activation/truncation in one layer == oracle conv -> add -> act."""
    rng = np.random.default_rng(k + cin * 3 + cout)
    n, h, w = nhw
    eps = 0.3
    pad = k // 2
    ctx, layer, rconv = _conv_layers(S, k, stride, pad, cin, cout, nhw, rng, act=pkg.ACT_RELU, eps=eps,
                                     n_in=2 if res else 1)
    radd, ract = orc.Add(S), orc.ActTrunc("relu", eps, S)
    oh, ow = layer.out_shape[1:3]
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    y0 = rconv.init(x0)
    # what the arithmetic leaves open, per element: the fp32 sum, and one unit in the last place of every
    # intermediate the two sides round independently (convolution sum; sum with the residual)
    sl0 = sum_slack(rconv, x0, bias=True) + ulp(y0, S)
    ins0 = [torch.from_numpy(x0).cuda()]
    if res:
        s0 = rng.normal(0, 1, (n, oh, ow, cout)).astype(NP_DTYPE[S])
        y0 = radd.init(y0, s0)
        sl0 = sl0 + ulp(y0, S)
        ins0.append(torch.from_numpy(s0).cuda())
    r0 = ract.init(y0)
    g0 = layer.init(ins0)
    ctx.sync()
    assert rel_err(to_np(g0), r0, slack=sl0) <= TOL[S]
    assert rel_err(to_np(layer.state_tensor(0)), ract.xA, slack=sl0) <= TOL[S]
    ties = 0
    for t, dens in enumerate([0.05, 0.3, 1.0, 0.0, 0.1]):
        # teacher forcing: the layer starts every frame from the oracle's state
        layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
        layer.state_tensor(1).copy_(torch.from_numpy(ract.xT).cuda())
        d = _rand_delta(rng, (n, h, w, cin), dens, S, 0.5)
        mid = rconv.step(d).poisoned()
        sl = sum_slack(rconv, d.zero_filled()) + ulp(mid.data, S)
        ins = [_upload(d)]
        if res:
            ds = _rand_delta(rng, (n, oh, ow, cout), dens / 2, S, 0.5)
            mid = radd.step(mid, ds).poisoned()
            sl = sl + ulp(mid.data, S)
            ins.append(_upload(ds))
        want = ract.step(mid).poisoned()
        out = layer.step(ins)
        ctx.sync()
        near = _near_tie(ract, eps, sl)
        ties += check_delta(out, want, S, f"fused frame {t}", allow_mask_diff=near, slack=sl)
        # state: equal to the oracle's where the decision agreed
        agree = to_np(out.mask) == want.mask
        assert rel_err(to_np(layer.state_tensor(0))[agree], ract.xA[agree], slack=sl[agree]) <= TOL[S]
        assert rel_err(to_np(layer.state_tensor(1))[agree], ract.xT[agree], slack=sl[agree]) <= TOL[S]
    assert ties <= 3


@pytest.mark.parametrize("S,k,cin,cout,nhw,res", [
    ("f16", 1, 64, 64, (2, 30, 30), False),       # wave-specialised kernel
    ("f16", 3, 32, 96, (1, 21, 24), True),        # three column blocks, residual
    ("f16", 3, 256, 256, (1, 12, 12), False),     # streamed weights: plain kernel tail
    ("f32", 3, 16, 32, (1, 20, 22), False),
    ("f16", 0, 0, 576, (2, 9, 11), False),        # k = 0: a stand-alone activation layer (wide pixels)
    ("f32", 0, 0, 2048, (1, 6, 6), False),        # eight vectors per lane: the pointer-addressed kernel
])
def test_layers_without_truncated_value_buffer(S, k, cin, cout, nhw, res):
    """no_xT = 1 (Section 6, memory remark): a truncated update is dropped, an update is x^A <- x^A + dx;
    teacher-forced against the oracle's ActTrunc(use_xT=False).  Buffer 1 does not exist."""
    rng = np.random.default_rng(k * 7 + cout)
    n, h, w = nhw
    eps = 1.6 if k else 0.3                                     # of the order of a pixel's largest change: both branches occur
    ract = orc.ActTrunc("relu", eps, S, use_xT=False)
    if k:
        wgt = (rng.normal(0, 1, (k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(NP_DTYPE[S])
        bias = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
        rconv, radd = orc.Conv(wgt, bias, 1, k // 2, False, S), orc.Add(S)
        ctx = pkg.Context(n * h * w)
        desc = pkg.make_desc(pkg.CONV, DT[S], n, h, w, cin, k=k, stride=1, pad=k // 2, cout=cout, act=pkg.ACT_RELU, eps=eps,
                             n_in=2 if res else 1, no_xT=1)
        layer = pkg.Layer(ctx, desc, torch.from_numpy(wgt).cuda(), torch.from_numpy(bias).cuda())
    else:
        cin = cout
        ctx = pkg.Context(n * h * w)
        layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, DT[S], n, h, w, cout, act=pkg.ACT_RELU, eps=eps, no_xT=1))
    with pytest.raises(pkg.DcnnError):
        layer.state_tensor(1)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    y0 = rconv.init(x0) if k else x0
    ins0 = [torch.from_numpy(x0).cuda()]
    if res:
        s0 = rng.normal(0, 1, (n, h, w, cout)).astype(NP_DTYPE[S])
        y0 = radd.init(y0, s0)
        ins0.append(torch.from_numpy(s0).cuda())
    r0 = ract.init(y0)
    g0 = layer.init(ins0)
    ctx.sync()
    sl0 = (sum_slack(rconv, x0, bias=True) + ulp(rconv.init(x0), S) + (ulp(y0, S) if res else 0.0)) if k else 0.0
    assert rel_err(to_np(g0), r0, slack=sl0) <= TOL[S]
    ties = 0
    saw_trunc = False
    for t, dens in enumerate([0.1, 0.5, 1.0, 0.0, 0.2]):
        layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
        d = _rand_delta(rng, (n, h, w, cin), dens, S, 0.05 if not k else 0.5)
        mid = rconv.step(d).poisoned() if k else d
        sl = (sum_slack(rconv, d.zero_filled()) + ulp(mid.data, S)) if k else np.zeros(mid.data.shape)
        ins = [_upload(d)]
        if res:
            ds = _rand_delta(rng, (n, h, w, cout), dens / 2, S, 0.5)
            mid = radd.step(mid, ds).poisoned()
            sl = sl + ulp(mid.data, S)
            ins.append(_upload(ds))
        xa_before = ract.xA.copy()
        want = ract.step(mid).poisoned()
        out = layer.step(ins)
        ctx.sync()
        near = _near_tie(ract, eps, sl)
        ties += check_delta(out, want, S, f"no-xT frame {t}", allow_mask_diff=near, exact_values=not k, slack=sl)
        agree = to_np(out.mask) == want.mask
        assert rel_err(to_np(layer.state_tensor(0))[agree], ract.xA[agree], slack=sl[agree]) <= TOL[S]
        trunc = (mid.mask == 1) & (want.mask == 0)
        saw_trunc |= bool(trunc.any())
        assert np.array_equal(ract.xA[trunc], xa_before[trunc])       # the oracle really dropped those updates
    assert ties <= 3 and (saw_trunc or cout > 96)


@pytest.mark.parametrize("S,k,cin,cin2,cout,nhw,stride2", [
    ("f16", 1, 64, 64, 256, (2, 24, 40), 1),
    ("f16", 1, 64, 32, 128, (1, 19, 23), 2),
    ("f16", 3, 32, 48, 64, (1, 33, 35), 1),
    ("f32", 1, 16, 8, 32, (1, 20, 20), 1),
    ("f32", 3, 16, 16, 32, (1, 17, 21), 2),
])
def test_conv_fused_projection(S, k, cin, cin2, cout, nhw, stride2):
    """conv_a(x) + conv_b(z) + activation/truncation in one layer (the 1x1 projection conv_b of the other
    arm of a residual add runs inside the same kernel) == oracle conv, conv, add, act."""
    rng = np.random.default_rng(7 * k + cin + cin2 + cout + stride2)
    n, oh, ow = nhw
    h, w = oh, ow                                           # main convolution: stride 1, same padding
    h2, w2 = (oh - 1) * stride2 + 1 + (stride2 - 1), (ow - 1) * stride2 + 1      # ragged: an unused last row
    if (h2 - 1) // stride2 + 1 != oh:
        h2 = (oh - 1) * stride2 + 1
    eps = 0.3
    wa = (rng.normal(0, 1, (k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(NP_DTYPE[S])
    wb = (rng.normal(0, 1, (1, 1, cin2, cout)) * np.sqrt(2.0 / cin2)).astype(NP_DTYPE[S])
    ba = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
    bb = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
    ra, rb = orc.Conv(wa, ba, 1, k // 2, False, S), orc.Conv(wb, bb, stride2, 0, False, S)
    radd, ract = orc.Add(S), orc.ActTrunc("relu", eps, S)
    ctx = pkg.Context(n * max(h * w, h2 * w2))
    desc = pkg.make_desc(pkg.CONV, DT[S], n, h, w, cin, k=k, stride=1, pad=k // 2, cout=cout, act=pkg.ACT_RELU, eps=eps,
                         n_in=2, proj=(cin2, h2, w2, stride2))
    wcat = torch.from_numpy(np.concatenate([wa.ravel(), wb.ravel()])).cuda()
    bcat = torch.from_numpy(np.concatenate([ba, bb])).cuda()
    layer = pkg.Layer(ctx, desc, wcat, bcat)
    assert layer.out_shape == (n, oh, ow, cout)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    z0 = rng.normal(0, 1, (n, h2, w2, cin2)).astype(NP_DTYPE[S])
    ya0, yb0 = ra.init(x0), rb.init(z0)
    y0 = radd.init(ya0, yb0)
    r0 = ract.init(y0)
    g0 = layer.init([torch.from_numpy(x0).cuda(), torch.from_numpy(z0).cuda()])
    ctx.sync()
    # both convolution sums and their sum are intermediates each side rounds on its own
    sl0 = sum_slack(ra, x0, bias=True) + sum_slack(rb, z0, bias=True) + ulp(ya0, S) + ulp(yb0, S) + ulp(y0, S)
    assert rel_err(to_np(g0), r0, slack=sl0) <= TOL[S], "dense first frame"
    assert rel_err(to_np(layer.state_tensor(0)), ract.xA, slack=sl0) <= TOL[S]
    ties = 0
    for t, (dx, dz) in enumerate([(0.05, 0.1), (0.3, 0.0), (0.0, 0.2), (1.0, 1.0), (0.0, 0.0), (0.1, 0.02)]):
        layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
        layer.state_tensor(1).copy_(torch.from_numpy(ract.xT).cuda())
        d = _rand_delta(rng, (n, h, w, cin), dx, S, 0.5)
        z = _rand_delta(rng, (n, h2, w2, cin2), dz, S, 0.5)
        ma, mb = ra.step(d).poisoned(), rb.step(z).poisoned()
        mid = radd.step(ma, mb).poisoned()
        sl = (sum_slack(ra, d.zero_filled()) + sum_slack(rb, z.zero_filled()) + ulp(ma.data, S) + ulp(mb.data, S)
              + ulp(mid.data, S))
        want = ract.step(mid).poisoned()
        out = layer.step([_upload(d), _upload(z)])
        ctx.sync()
        near = _near_tie(ract, eps, sl)
        ties += check_delta(out, want, S, f"projection frame {t}", allow_mask_diff=near, slack=sl)
        agree = to_np(out.mask) == want.mask
        assert rel_err(to_np(layer.state_tensor(0))[agree], ract.xA[agree], slack=sl[agree]) <= TOL[S]
        assert rel_err(to_np(layer.state_tensor(1))[agree], ract.xT[agree], slack=sl[agree]) <= TOL[S]
        st = layer.stats()
        assert st["pixels_in"] == d.count and st["pixels_in2"] == z.count and st["pixels_work"] == mid.count
    assert ties <= 3


@pytest.mark.parametrize("S,k,cin,cout,nhw,proj", [
    ("f16", 1, 64, 256, (2, 24, 40), True),
    ("f16", 3, 32, 64, (1, 33, 35), False),
    ("f32", 1, 16, 32, (1, 20, 21), False),
    ("f32", 3, 16, 32, (1, 17, 21), True),
])
def test_conv_fused_accumulate(S, k, cin, cout, nhw, proj):
    """The network's output layer folded into the last convolution + activation: the layer keeps the dense
    accumulated output O and adds every emitted delta to it == oracle conv (, conv, add), act, accumulate."""
    rng = np.random.default_rng(11 * k + cin + cout + int(proj))
    n, h, w = nhw
    cin2 = 16
    eps = 0.3
    wa = (rng.normal(0, 1, (k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(NP_DTYPE[S])
    wb = (rng.normal(0, 1, (1, 1, cin2, cout)) * np.sqrt(2.0 / cin2)).astype(NP_DTYPE[S])
    ba = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
    bb = rng.normal(0, 0.1, cout).astype(NP_DTYPE[S])
    ra, rb = orc.Conv(wa, ba, 1, k // 2, False, S), orc.Conv(wb, bb, 1, 0, False, S)
    radd, ract, racc = orc.Add(S), orc.ActTrunc("relu", eps, S), orc.Accumulate(S)
    ctx = pkg.Context(n * h * w)
    desc = pkg.make_desc(pkg.CONV, DT[S], n, h, w, cin, k=k, stride=1, pad=k // 2, cout=cout, act=pkg.ACT_RELU, eps=eps,
                         n_in=2 if proj else 1, proj=(cin2, h, w, 1) if proj else None, fuse_accum=1, want_idx=0)
    wcat = np.concatenate([wa.ravel(), wb.ravel()]) if proj else wa
    bcat = np.concatenate([ba, bb]) if proj else ba
    layer = pkg.Layer(ctx, desc, torch.from_numpy(wcat).cuda(), torch.from_numpy(bcat).cuda())
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(NP_DTYPE[S])
    z0 = rng.normal(0, 1, (n, h, w, cin2)).astype(NP_DTYPE[S])
    y0 = ra.init(x0)
    sl0 = sum_slack(ra, x0, bias=True) + ulp(y0, S)
    if proj:
        yb0 = rb.init(z0)
        y0 = radd.init(y0, yb0)
        sl0 = sl0 + sum_slack(rb, z0, bias=True) + ulp(yb0, S) + ulp(y0, S)
    r0 = racc.init(ract.init(y0))
    g0 = layer.init([torch.from_numpy(x0).cuda()] + ([torch.from_numpy(z0).cuda()] if proj else []))
    ctx.sync()
    assert rel_err(to_np(g0), r0, slack=sl0) <= TOL[S]
    assert np.array_equal(to_np(layer.state_tensor(2)), to_np(g0)), "O starts as the dense first output"
    for t, dens in enumerate([0.05, 0.3, 1.0, 0.0, 0.1]):
        layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
        layer.state_tensor(1).copy_(torch.from_numpy(ract.xT).cuda())
        layer.state_tensor(2).copy_(torch.from_numpy(racc.O).cuda())
        d = _rand_delta(rng, (n, h, w, cin), dens, S, 0.5)
        mid = ra.step(d).poisoned()
        sl = sum_slack(ra, d.zero_filled()) + ulp(mid.data, S)
        ins = [_upload(d)]
        if proj:
            z = _rand_delta(rng, (n, h, w, cin2), dens / 2, S, 0.5)
            mb = rb.step(z).poisoned()
            mid = radd.step(mid, mb).poisoned()
            sl = sl + sum_slack(rb, z.zero_filled()) + ulp(mb.data, S) + ulp(mid.data, S)
            ins.append(_upload(z))
        o_before = racc.O.copy()
        want = ract.step(mid).poisoned()
        o_ref = racc.step(want)
        out = layer.step(ins)
        ctx.sync()
        gm = to_np(out.mask)
        near = _near_tie(ract, eps, sl)
        assert np.all(near[gm != want.mask]), f"frame {t}: mask mismatch away from a threshold tie"
        agree = gm == want.mask
        got_o = to_np(layer.state_tensor(2)).reshape(o_ref.shape)
        assert not np.isnan(got_o.astype(np.float64)).any()
        # the folded layer writes O = f(new x^A), the oracle's output layer adds the rounded delta onto O:
        # one more independent rounding, of the delta
        sl_o = sl + ulp(want.data, S)
        assert rel_err(got_o[agree], o_ref[agree], slack=sl_o[agree]) <= TOL[S], f"frame {t}: accumulated output"
        untouched = want.mask == 0
        assert np.array_equal(got_o[untouched & agree], o_before[untouched & agree]), "O changes only where a delta was emitted"
        assert out.data.data_ptr() == layer.state_tensor(2).data_ptr(), "the layer's output data is O"


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("stride,c", [(1, 32), (2, 192), (1, 960), (2, 20)])
def test_depthwise(S, stride, c):
    rng = np.random.default_rng(stride + c)
    nhw = (1, 28, 27)
    eps = 0.3
    ctx, layer, rconv = _conv_layers(S, 3, stride, 1, c, c, nhw, rng, act=pkg.ACT_RELU6, eps=eps, depthwise=True)
    ract = orc.ActTrunc("relu6", eps, S)
    x0 = rng.normal(0, 1, nhw + (c,)).astype(NP_DTYPE[S])
    y0 = rconv.init(x0)
    r0 = ract.init(y0)
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert rel_err(to_np(g0), r0, slack=sum_slack(rconv, x0, bias=True) + ulp(y0, S)) <= TOL[S]
    ties = 0
    for t, dens in enumerate([0.1, 0.5, 0.0]):
        layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
        layer.state_tensor(1).copy_(torch.from_numpy(ract.xT).cuda())
        d = _rand_delta(rng, nhw + (c,), dens, S, 0.5)
        mid = rconv.step(d).poisoned()
        sl = sum_slack(rconv, d.zero_filled()) + ulp(mid.data, S)
        want = ract.step(mid).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        near = _near_tie(ract, eps, sl)
        ties += check_delta(out, want, S, f"depthwise frame {t}", allow_mask_diff=near, slack=sl)
    assert ties <= 3


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("k,stride,pad,what", [(1, 1, 0, "batchnorm"), (2, 2, 0, "avgpool"), (3, 2, 1, "avgpool")])
def test_depthwise_as_batchnorm_and_average_pooling(S, k, stride, pad, what):
    """The remaining linear per-channel layers are depthwise convolutions: an unfused batch norm is a 1x1
    depthwise layer (scale on the delta, shift only in the first frame -- Section 3.1: biases enter once),
    average pooling a k x k depthwise layer with weights 1/k^2 (zero padding counted)."""
    rng = np.random.default_rng(k * 10 + stride)
    n, h, w, c = 2, 26, 22, 48
    if what == "batchnorm":
        wgt = rng.uniform(0.5, 1.5, (1, 1, c)).astype(NP_DTYPE[S])
        bias = rng.normal(0, 0.5, c).astype(NP_DTYPE[S])
    else:
        wgt = np.full((k, k, c), 1.0 / (k * k)).astype(NP_DTYPE[S])
        bias = np.zeros(c, NP_DTYPE[S])
    ref = orc.Conv(wgt, bias, stride, pad, True, S)
    ctx = pkg.Context(n * h * w)
    desc = pkg.make_desc(pkg.DWCONV, DT[S], n, h, w, c, k=k, stride=stride, pad=pad, cout=c)
    layer = pkg.Layer(ctx, desc, torch.from_numpy(wgt).cuda(), torch.from_numpy(bias).cuda())
    x0 = rng.normal(0, 1, (n, h, w, c)).astype(NP_DTYPE[S])
    r0 = ref.init(x0)
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert rel_err(to_np(g0), r0, slack=sum_slack(ref, x0, bias=True)) <= TOL[S]
    for t, dens in enumerate([0.1, 0.6, 0.0]):
        d = _rand_delta(rng, (n, h, w, c), dens, S)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"{what} frame {t}", slack=sum_slack(ref, d.zero_filled()))


# ---- pooling, upsampling, accumulation (bit-exact) -----------------------------------------------
@pytest.mark.parametrize("S", ["f32", "f16"])
def test_maxpool(S):
    rng = np.random.default_rng(3)
    shape = (2, 33, 30, 64)
    n, h, w, c = shape
    ref = orc.MaxPool(3, 2, 1, S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.MAXPOOL, DT[S], n, h, w, c, k=3, stride=2, pad=1))
    x0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    r0 = ref.init(x0)
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), r0)
    for t, dens in enumerate([0.1, 0.6, 0.0]):
        d = _rand_delta(rng, shape, dens, S, 0.7)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"maxpool frame {t}", exact_values=True)
        assert np.array_equal(to_np(layer.state_tensor(0)), ref.xA)


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("factor", [2, 4])
def test_upsample(S, factor):
    rng = np.random.default_rng(factor)
    shape = (2, 9, 12, 32)
    n, h, w, c = shape
    ref = orc.Upsample(factor, S)
    ctx = pkg.Context(n * h * w * factor * factor)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.UPSAMPLE, DT[S], n, h, w, c, factor=factor))
    x0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), ref.init(x0))
    for t, dens in enumerate([0.1, 1.0, 0.0]):
        d = _rand_delta(rng, shape, dens, S)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"upsample frame {t}", exact_values=True)


@pytest.mark.parametrize("n,h,w,factor", [(1, 100, 102, 2), (1, 101, 102, 2), (2, 70, 81, 2), (1, 66, 103, 3), (1, 67, 103, 3), (1, 64, 64, 4)])
def test_upsampled_mask_on_both_sides_of_the_one_launch_list(n, h, w, factor):
    """Input pixels x factor just below and above 20 K: the list in one launch and in two passes, values and mask bit for bit."""
    S, shape = "f16", (n, h, w, 8)
    rng = np.random.default_rng(h * factor)
    ref = orc.Upsample(factor, S)
    ctx = pkg.Context(n * h * w * factor * factor)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.UPSAMPLE, DT[S], n, h, w, 8, factor=factor))
    x0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    layer.init([torch.from_numpy(x0).cuda()])
    ref.init(x0)
    for t, dens in enumerate([0.3, 0.0, 1.0, 0.05]):
        d = _rand_delta(rng, shape, dens, S)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"upsample x{factor} frame {t}", exact_values=True)


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("factor,c", [(2, 32), (3, 5), (4, 16)])
def test_upsample_bilinear(S, factor, c):
    """Masks and lists bit-exact (integer tap rule); values within tolerance (fp32 weights vs float64)."""
    rng = np.random.default_rng(factor * 10 + c)
    shape = (2, 7, 9, c)
    n, h, w, _ = shape
    ref = orc.UpsampleBilinear(factor, S)
    ctx = pkg.Context(n * h * w * factor * factor)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.UPSAMPLE_BILINEAR, DT[S], n, h, w, c, factor=factor))
    assert layer.out_shape == (n, h * factor, w * factor, c)
    x0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    # a weighted sum of up to four sources in fp32 against the oracle's float64: same allowance as a convolution sum
    mag = orc.UpsampleBilinear(factor, "f64")
    assert rel_err(to_np(g0), ref.init(x0), slack=8 * U32 * mag.init(np.abs(x0))) <= TOL[S]
    for t, dens in enumerate([0.1, 1.0, 0.02, 0.0]):
        d = _rand_delta(rng, shape, dens, S)
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"bilinear x{factor} frame {t}", slack=8 * U32 * mag.init(np.abs(d.zero_filled())))


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("shape", [(3, 7, 7, 64), (2, 13, 10, 20), (5, 4, 6, 3), (1, 1, 1, 8), (2, 24, 24, 1280)])
def test_global_average_pooling(S, shape):
    rng = np.random.default_rng(sum(shape))
    n, h, w, c = shape
    ref = orc.GlobalAvgPool(S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.GAVGPOOL, DT[S], n, h, w, c))
    assert layer.out_shape == (n, 1, 1, c)
    x0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    g0 = layer.init([torch.from_numpy(x0).cuda()])
    ctx.sync()
    mag = orc.GlobalAvgPool("f64")
    assert rel_err(to_np(g0), ref.init(x0), slack=8 * U32 * mag.init(np.abs(x0))) <= TOL[S]
    for t, dens in enumerate([0.1, 1.0, 0.0]):
        d = _rand_delta(rng, shape, dens, S)
        if t == 0 and n > 1:
            d.mask[1] = 0                                       # one stream without any update
            d.data[1] = np.nan
        want = ref.step(d).poisoned()
        out = layer.step([_upload(d)])
        ctx.sync()
        check_delta(out, want, S, f"global average pool frame {t}",
                    slack=8 * U32 * mag.init(np.abs(d.zero_filled().astype(np.float64))))


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("ca,cb", [(32, 64), (16, 3), (5, 7)])
def test_concat(S, ca, cb):
    """Channel concatenation: values are copies (bit-exact); an unflagged stream contributes zeros."""
    rng = np.random.default_rng(ca * 100 + cb)
    n, h, w = 2, 23, 19
    ref = orc.Concat(S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.CONCAT, DT[S], n, h, w, ca, cout=ca + cb, n_in=2))
    assert layer.out_shape == (n, h, w, ca + cb)
    a0 = rng.normal(0, 1, (n, h, w, ca)).astype(NP_DTYPE[S])
    b0 = rng.normal(0, 1, (n, h, w, cb)).astype(NP_DTYPE[S])
    g0 = layer.init([torch.from_numpy(a0).cuda(), torch.from_numpy(b0).cuda()])
    ctx.sync()
    assert np.array_equal(to_np(g0), ref.init(a0, b0))
    for t, (da_, db_) in enumerate([(0.2, 0.1), (1.0, 0.0), (0.0, 0.3), (0.0, 0.0)]):
        da = _rand_delta(rng, (n, h, w, ca), da_, S)
        db = _rand_delta(rng, (n, h, w, cb), db_, S)
        want = ref.step(da, db).poisoned()
        out = layer.step([_upload(da), _upload(db)])
        ctx.sync()
        check_delta(out, want, S, f"concat frame {t}", exact_values=True)


@pytest.mark.parametrize("S", ["f32", "f16"])
def test_accumulate(S):
    rng = np.random.default_rng(8)
    shape = (2, 21, 19, 256)
    n, h, w, c = shape
    ref = orc.Accumulate(S)
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACCUM, DT[S], n, h, w, c))
    y0 = rng.normal(0, 1, shape).astype(NP_DTYPE[S])
    ref.init(y0)
    layer.init([torch.from_numpy(y0).cuda()])
    for t, dens in enumerate([0.1, 0.7, 0.0]):
        d = _rand_delta(rng, shape, dens, S)
        want = ref.step(d)
        out = layer.step([_upload(d)])
        ctx.sync()
        assert np.array_equal(to_np(out.data), want)


# ---- error paths through the ABI ------------------------------------------------------------------
def test_error_paths():
    ctx = pkg.Context(16 * 16)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.ACT, pkg.F32, 1, 16, 16, 8, act=pkg.ACT_RELU, eps=0.1))
    d = _upload(ODelta(np.zeros((1, 16, 16, 8), np.float32), np.zeros((1, 16, 16), np.uint8)))
    with pytest.raises(pkg.DcnnError) as e:
        layer.step([d])                                   # step before the first frame
    assert e.value.status == 4
    layer.init([torch.zeros((1, 16, 16, 8), device="cuda")])
    bad = _upload(ODelta(np.zeros((1, 8, 16, 8), np.float32), np.zeros((1, 8, 16), np.uint8)))
    with pytest.raises(pkg.DcnnError) as e:
        layer.step([bad])
    assert e.value.status == 2
    half = _upload(ODelta(np.zeros((1, 16, 16, 8), np.float16), np.zeros((1, 16, 16), np.uint8)))
    with pytest.raises(pkg.DcnnError) as e:
        layer.step([half])
    assert e.value.status == 3
    layer.reset()
    with pytest.raises(pkg.DcnnError):
        layer.step([d])
    small = pkg.Context(64)                               # workspace too small for this layer
    l2 = pkg.Layer(small, pkg.make_desc(pkg.ACT, pkg.F32, 1, 64, 64, 8, act=pkg.ACT_RELU, eps=0.1, n_in=2))
    l2.init([torch.zeros((1, 64, 64, 8), device="cuda")] * 2)
    big = _upload(ODelta(np.zeros((1, 64, 64, 8), np.float32), np.zeros((1, 64, 64), np.uint8)))
    with pytest.raises(pkg.DcnnError) as e:
        l2.step([big, big])
    assert e.value.status == 5
    with pytest.raises(pkg.DcnnError) as e:               # a fused activation needs the whole pixel in one LDS tile
        pkg.Layer(ctx, pkg.make_desc(pkg.CONV, pkg.F16, 1, 16, 16, 64, k=1, stride=1, pad=0, cout=2048,
                                     act=pkg.ACT_RELU, eps=0.1),
                  torch.zeros((1, 1, 64, 2048), dtype=torch.float16, device="cuda"))
    assert e.value.status == 7


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,mode", [
    ("f16", 1, 1, 64, 64, (1, 8, 9), "plain"),           # 72 pixels: a tile and a remainder of 8
    ("f16", 3, 1, 64, 200, (3, 17, 13), "act"),          # channel tile remainder, pixels over stream borders
    ("f16", 3, 2, 256, 136, (2, 15, 15), "residual"),    # K-steps split over the waves, odd stride-2 border
    ("f32", 3, 1, 64, 64, (1, 16, 5), "act"),            # fp32, split
    ("f32", 7, 2, 8, 12, (1, 21, 19), "plain"),          # wide window, 12 channels
    ("f16", 1, 1, 32, 256, (2, 12, 11), "projection"),   # second K loop, four channel tiles side by side
    ("f32", 1, 1, 16, 64, (1, 9, 31), "projection"),
    ("f16", 1, 1, 24, 32, (2, 20, 21), "act"),           # tiles of 32 channels, whole and split sums, a projection
    ("f32", 3, 1, 24, 20, (2, 11, 13), "residual"),
    ("f16", 1, 1, 48, 24, (2, 9, 14), "projection"),
    ("f16", 1, 1, 16, 320, (3, 17, 23), "act"),          # five channel tiles, one wave each, pixel groups no multiple of the XCDs
    ("f16", 3, 1, 128, 72, (4, 92, 94), "act"),          # batch on the plain kernel, a single stream on tiles
])
def test_first_frame_tiles(S, k, stride, cin, cout, nhw, mode):
    """The dense first frame at the edges of its tiles (64 pixels x 64 channels, with and without split K), and the same
    bits for a stream alone as in the batch."""
    n, h, w = nhw
    pad = k // 2
    rng = np.random.default_rng(91)
    dt = NP_DTYPE[S]
    wgt = (rng.standard_normal((k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(dt)
    bias = rng.normal(0, 0.5, cout).astype(dt)
    x = rng.standard_normal((n, h, w, cin)).astype(dt)
    conv = orc.Conv(wgt, bias, stride, pad, False, S)
    y = np.asarray(conv.init(x))
    slack = sum_slack(conv, x, bias=True) + ulp(y, S)
    oh, ow = y.shape[1:3]
    second, w2, b2, proj = [], [], [], None
    if mode == "residual":
        second = [rng.standard_normal(y.shape).astype(dt)]
        y = (y.astype(np.float64) + second[0].astype(np.float64)).astype(dt)
    elif mode == "projection":
        second = [rng.standard_normal((n, oh, ow, 24)).astype(dt)]
        pw = (rng.standard_normal((1, 1, 24, cout)) * np.sqrt(2.0 / 24)).astype(dt)
        pb = rng.normal(0, 0.5, cout).astype(dt)
        pc = orc.Conv(pw, pb, 1, 0, False, S)
        z = np.asarray(pc.init(second[0]))
        slack = slack + sum_slack(pc, second[0], bias=True) + ulp(z, S)
        y = (y.astype(np.float64) + z.astype(np.float64)).astype(dt)
        w2, b2, proj = [pw.reshape(-1)], [pb], (24, oh, ow, 1)
    act = "none" if mode == "plain" else "relu"
    slack = slack + ulp(y, S)

    def run(streams):
        m = len(streams)
        ctx = pkg.Context(m * max(h * w, oh * ow))
        layer = pkg.Layer(ctx, pkg.make_desc(pkg.CONV, DT[S], m, h, w, cin, k=k, stride=stride, pad=pad, cout=cout,
                                             act=pkg.ACT_RELU if act == "relu" else pkg.ACT_NONE, eps=0.05, n_in=1 + len(second), proj=proj),
                          torch.from_numpy(np.concatenate([wgt.reshape(-1)] + w2)).cuda(),
                          torch.from_numpy(np.concatenate([bias] + b2)).cuda())
        out = layer.init([torch.from_numpy(np.ascontiguousarray(a[streams])).cuda() for a in [x] + second])
        ctx.sync()
        state = [to_np(layer.state_tensor(i)) for i in (0, 1)] if act == "relu" else []
        return to_np(out), state

    got, state = run(list(range(n)))
    ref = np.maximum(y, dt(0)) if act == "relu" else y
    assert rel_err(got, ref, slack=slack) <= TOL[S]
    if act == "relu":
        assert rel_err(state[0], y, slack=slack) <= TOL[S]
        assert not state[1].any()
    alone, _ = run([n - 1])
    assert np.array_equal(alone[0], got[n - 1])


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,mode", [
    ("f16", 1, 1, 40, 64, (1, 9, 7), "act"),             # lines of 128 bytes: part of one, a whole one and a part, four and a part
    ("f16", 3, 1, 72, 40, (2, 10, 11), "plain"),
    ("f16", 1, 1, 264, 64, (1, 9, 13), "residual"),
    ("f32", 3, 2, 36, 32, (1, 13, 12), "act"),
    ("f16", 3, 1, 32, 96, (2, 9, 14), "act"),            # rows of up to 64 bytes, whole and split sums
    ("f16", 5, 1, 24, 32, (1, 8, 9), "plain"),
    ("f16", 3, 1, 16, 64, (2, 9, 14), "act"),            # up to 32: four taps together, whole and split sums
    ("f32", 3, 2, 4, 20, (1, 11, 12), "plain"),
    ("f16", 7, 1, 8, 72, (1, 9, 8), "act"),
    ("f16", 3, 1, 24, 40, (2, 13, 15), "act"),           # windows whose last K-step of two or three is half empty, whole and split sums
    ("f16", 3, 2, 40, 64, (1, 15, 14), "plain"),
    ("f16", 5, 1, 40, 24, (1, 8, 9), "residual"),
    ("f16", 7, 1, 24, 72, (1, 9, 8), "act"),
    ("f16", 1, 1, 24, 200, (1, 70, 61), "act"),          # tiles of 32 channels on small maps: whole sums, a last tile of 8, and beyond
    ("f16", 1, 1, 24, 256, (4, 64, 64), "projection"),   # them 1024 tiles of 64, which are split too
    ("f32", 3, 1, 40, 72, (1, 50, 41), "residual"),
])
def test_first_frame_lines_of_a_pixel(S, k, stride, cin, cout, nhw, mode):
    """How the first frame's kernel fetches a pixel's channels: by quads of lanes, or a pixel per lane, at the ends of its groups."""
    test_first_frame_tiles(S, k, stride, cin, cout, nhw, mode)


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,mode", [
    # 2048 tiles of 64 pixels x 64 channels: the batch on tiles of 64 channels, a stream alone on tiles of 32, whole sums
    ("f16", 1, 1, 24, 256, (8, 64, 64), "projection"),   # one line of two K-steps, for the projection too
    ("f16", 1, 1, 72, 256, (8, 64, 65), "projection"),   # a line and a part
    ("f16", 1, 1, 128, 256, (8, 64, 64), "residual"),    # whole lines
    ("f16", 3, 1, 32, 64, (8, 127, 130), "act"),         # one line of two K-steps over a window
    ("f32", 1, 1, 40, 256, (8, 64, 64), "residual"),
    # ... of which every lane fetches its own pixel
    ("f16", 3, 1, 16, 64, (8, 128, 128), "residual"),
    ("f16", 3, 1, 24, 64, (8, 128, 129), "act"),
    ("f16", 1, 1, 40, 256, (8, 64, 64), "residual"),     # wide layers over broken lines
    ("f16", 3, 1, 72, 256, (8, 64, 64), "plain"),
    ("f16", 1, 1, 56, 64, (9, 121, 128), "act"),         # one round of three workgroups per compute unit
    ("f16", 1, 1, 88, 512, (1, 30, 41), "plain"),        # (tiles of 32: few pixels)
    # padded lines: split sums over 3x3, over any window with few tiles, fp32; whole sums of one workgroup per compute unit
    ("f16", 3, 1, 72, 64, (4, 40, 41), "act"),
    ("f16", 5, 1, 88, 40, (1, 20, 21), "plain"),
    ("f32", 3, 1, 100, 64, (2, 21, 20), "residual"),
    ("f16", 3, 1, 96, 384, (1, 80, 76), "act"),
])
def test_first_frame_tile_widths_and_fetches(S, k, stride, cin, cout, nhw, mode):
    """Both widths of a tile and both ways to fetch a pixel, on both sides of the rules that choose them."""
    test_first_frame_tiles(S, k, stride, cin, cout, nhw, mode)


def test_first_frame_of_a_batch_past_2_gib_has_the_bits_of_single_streams():
    """3x3 64->16 on 112x112 with its K-steps split over four waves: 1400 streams hold 2.09 GiB of input (two launches); the first,
    the one at the border of the launches and the last stream against the same streams alone."""
    n, h, w, cin, cout = 1400, 112, 112, 64, 16
    torch.manual_seed(5)
    x = torch.randn((n, h, w, cin), dtype=torch.float16, device="cuda")
    assert x.numel() * 2 > 2 ** 31
    wgt = (torch.randn((3, 3, cin, cout), device="cuda") * 0.06).half()

    def run(streams):
        m = streams.shape[0]
        ctx = pkg.Context(m * h * w)
        layer = pkg.Layer(ctx, pkg.make_desc(pkg.CONV, pkg.F16, m, h, w, cin, k=3, pad=1, cout=cout, act=pkg.ACT_RELU, eps=0.05), wgt)
        out = layer.init([streams])
        ctx.sync()
        return out, layer.state_tensor(0), layer

    out, buf, _keep = run(x)
    border = (2 ** 31 - 1) // (h * w * cin * 2)
    for i in (0, border - 1, border, n - 1):
        alone, alone_buf, _keep2 = run(x[i:i + 1].contiguous())
        assert torch.equal(out[i], alone[0]) and torch.equal(buf[i], alone_buf[0]), f"stream {i}"


@pytest.mark.parametrize("S", ["f32", "f16"])
@pytest.mark.parametrize("k,stride,c,hw", [(3, 1, 16, (5, 7)), (3, 2, 200, (9, 6)), (2, 2, 8, (6, 6)), (1, 1, 24, (3, 1))])
def test_depthwise_first_frame_pixel_groups(S, k, stride, c, hw):
    """Four neighbouring pixels of the flat order per thread: groups that straddle rows and streams, and the last one."""
    n, (h, w), pad = 3, hw, k // 2 if k == 3 else 0
    rng = np.random.default_rng(17)
    dt = NP_DTYPE[S]
    wgt = rng.standard_normal((k, k, c)).astype(dt)
    bias = rng.normal(0, 0.5, c).astype(dt)
    x = rng.standard_normal((n, h, w, c)).astype(dt)
    conv = orc.Conv(wgt, bias, stride, pad, True, S)
    y = np.asarray(conv.init(x))
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.DWCONV, DT[S], n, h, w, c, k=k, stride=stride, pad=pad, cout=c,
                                         act=pkg.ACT_RELU6, eps=0.05), torch.from_numpy(wgt).cuda(), torch.from_numpy(bias).cuda())
    out = layer.init([torch.from_numpy(x).cuda()])
    ctx.sync()
    slack = sum_slack(conv, x, bias=True) + ulp(y, S)
    assert rel_err(to_np(out), np.clip(y, dt(0), dt(6)), slack=slack) <= TOL[S]
    assert rel_err(to_np(layer.state_tensor(0)), y, slack=slack) <= TOL[S]


@pytest.mark.parametrize("n,h,w", [(1, 1, 1), (2, 9, 9), (1, 3, 31), (3, 33, 18), (4, 128, 128), (1, 257, 255), (5, 64, 205)])
@pytest.mark.parametrize("k,stride,pad", [(1, 1, 0), (1, 2, 0), (3, 1, 1), (3, 2, 1)])
@pytest.mark.parametrize("second", [False, True])
def test_mask_compact_on_words_of_flags(n, h, w, k, stride, pad, second):
    """Maps whose rows, words of 32 flags and streams do not line up, up to and just past the 64 K pixels that one launch
    serves (4 x 128 x 128 = 65536; 257 x 255 = 65535; 5 x 64 x 205 = 65600)."""
    rng = np.random.default_rng(n * 1000 + w)
    mask = (rng.random((n, h, w)) < 0.07).astype(np.uint8)
    mask[:, 0, 0] = mask[:, -1, -1] = 1
    want = orc.window_mask(mask, k, stride, pad)
    mask_b = (rng.random(want.shape) < 0.03).astype(np.uint8) if second else None
    if second:
        want = want | mask_b
    ctx = pkg.Context(n * h * w)
    got, idx, count = ctx.mask_compact(torch.from_numpy(mask).cuda(), k, stride, pad, torch.from_numpy(mask_b).cuda() if second else None)
    ctx.sync()
    assert np.array_equal(to_np(got), want)
    flat = np.flatnonzero(want.reshape(-1))
    assert int(to_np(count)[0]) == flat.size
    assert np.array_equal(to_np(idx)[:flat.size], flat)


@pytest.mark.parametrize("n,h,w", [(1, 5, 9), (3, 37, 53), (40, 9, 7), (2, 96, 130), (1, 3, 9000), (1, 12, 8000)])
@pytest.mark.parametrize("k,stride,pad", [(5, 1, 2), (7, 2, 3), (5, 2, 0), (7, 1, 6), (9, 1, 4)])
def test_mask_compact_wide_windows(n, h, w, k, stride, pad):
    """Windows from 5x5 on: chunks that start and end within rows, cross several streams, and (8000 wide) runs of input
    flags that do not fit a workgroup's room."""
    if h + 2 * pad < k or w + 2 * pad < k:
        pytest.skip("window larger than the map")
    rng = np.random.default_rng(n + h + w)
    mask = (rng.random((n, h, w)) < 0.01).astype(np.uint8)
    mask[:, -1, 0] = 1
    want = orc.window_mask(mask, k, stride, pad)
    ctx = pkg.Context(max(mask.size, want.size))
    got, idx, count = ctx.mask_compact(torch.from_numpy(mask).cuda(), k, stride, pad)
    ctx.sync()
    assert np.array_equal(to_np(got), want)
    flat = np.flatnonzero(want.reshape(-1))
    assert int(to_np(count)[0]) == flat.size
    assert np.array_equal(to_np(idx)[:flat.size], flat)


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,res", [
    ("f16", 3, 1, 256, 512, (2, 8, 9), False),       # whole groups of K-steps, 16 channel blocks
    ("f16", 1, 1, 520, 776, (3, 7, 11), False),      # a K-step past the pixel's channels, a block of 8 channels
    ("f16", 3, 2, 136, 1032, (1, 13, 15), False),    # nine K-steps per tap, stride 2 on odd sizes
    ("f16", 1, 1, 1024, 512, (2, 5, 6), True),       # residual without an activation
    ("f32", 3, 1, 132, 260, (1, 9, 10), False),
    ("f32", 1, 2, 512, 516, (2, 12, 7), False),
])
def test_conv_per_channel_block(S, k, stride, cin, cout, nhw, res):
    """Weights too large for LDS on a small map, no activation: a wave per (tile, 32 channels)."""
    n, h, w = nhw
    pad = k // 2
    rng = np.random.default_rng(cin + cout)
    dt = NP_DTYPE[S]
    wgt = (rng.standard_normal((k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(dt)
    conv = orc.Conv(wgt, None, stride, pad, False, S)
    x0 = np.zeros((n, h, w, cin), dt)
    y0 = np.asarray(conv.init(x0))
    ctx = pkg.Context(n * h * w)
    layer = pkg.Layer(ctx, pkg.make_desc(pkg.CONV, DT[S], n, h, w, cin, k=k, stride=stride, pad=pad, cout=cout, n_in=2 if res else 1),
                      torch.from_numpy(wgt).cuda(), None)
    layer.init([torch.from_numpy(a).cuda() for a in [x0] + ([np.zeros_like(y0)] if res else [])])
    for dens in (0.05, 0.6, 1.0, 0.0):
        d = _rand_delta(rng, (n, h, w, cin), dens, S)
        want = conv.step(d)
        slack = sum_slack(conv, d.zero_filled())
        ins = [_upload(d)]
        if res:
            r = _rand_delta(rng, y0.shape, 0.4, S)
            ins.append(_upload(r))
            base = np.where(want.mask[..., None] == 1, np.nan_to_num(want.data), dt(0))
            total = (base.astype(np.float64) + r.zero_filled().astype(np.float64)).astype(dt)
            slack = slack + ulp(base, S)
            want = ODelta(total, want.mask | r.mask)
        out = layer.step(ins)
        ctx.sync()
        check_delta(out, want.poisoned(), S, f"density {dens}", slack=slack)


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw,res", [
    ("f16", 3, 1, 72, 392, (3, 40, 41), False),      # four waves to a tile, the last of 13 channel blocks alone; a line and a part
    ("f16", 3, 1, 72, 392, (1, 50, 51), False),      # two waves, each for itself
    ("f16", 1, 1, 520, 1048, (2, 32, 37), True),     # four, nine lines with a residual
    ("f16", 1, 1, 1552, 264, (1, 9, 10), False),     # one, a long sum
])
def test_conv_per_channel_block_with_shared_operands(S, k, stride, cin, cout, nhw, res):
    """fp16 units whose waves share the gathered operands of their tile."""
    test_conv_per_channel_block(S, k, stride, cin, cout, nhw, res)


@pytest.mark.parametrize("S,kind,k,stride,cin,cout,nhw", [
    ("f16", "conv", 3, 1, 32, 32, (1, 20, 23)),          # resident weights
    ("f16", "conv", 3, 2, 64, 128, (2, 21, 18)),
    ("f16", "conv", 3, 1, 256, 256, (1, 14, 15)),        # streamed weights
    ("f32", "conv", 5, 1, 12, 20, (1, 17, 16)),          # plain kernel
    ("f16", "dwconv", 3, 1, 96, 96, (2, 13, 17)),
    ("f16", "add", 1, 1, 64, 64, (1, 19, 31)),
    ("f16", "add", 1, 1, 1024, 1024, (1, 11, 13)),
])
def test_a_captured_step_of_a_layer_with_its_own_list_replays(S, kind, k, stride, cin, cout, nhw):
    """One step recorded into a graph and replayed on changing inputs: each replay leaves mask, values and buffers of the same
    step of an eager layer -- in particular no flag of an earlier replay."""
    n, h, w = nhw
    rng = np.random.default_rng(cin + h)
    dt, n_in = NP_DTYPE[S], 2 if kind == "add" else 1
    code = {"conv": pkg.CONV, "dwconv": pkg.DWCONV, "add": pkg.ACT}[kind]
    desc = pkg.make_desc(code, DT[S], n, h, w, cin, k=k, stride=stride, pad=k // 2, cout=cout, act=pkg.ACT_RELU, eps=0.3, n_in=n_in, want_idx=0)
    wgt = None if kind == "add" else torch.from_numpy((rng.standard_normal((k, k, cin, cout) if kind == "conv" else (k, k, cin)) *
                                                       np.sqrt(2.0 / (k * k * (cin if kind == "conv" else 1)))).astype(dt)).cuda()
    dense = [torch.from_numpy(rng.standard_normal((n, h, w, cin)).astype(dt)).cuda() for _ in range(n_in)]
    frames = [[_rand_delta(rng, (n, h, w, cin), dens, S, 0.4) for _ in range(n_in)] for dens in (0.02, 0.3, 1.0, 0.0, 0.03, 0.0, 0.5)]
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = pkg.Context(n * h * w)
        eager, replayed = (pkg.Layer(ctx, desc, wgt) for _ in range(2))
        fixed = [pkg.Delta(torch.zeros_like(d), torch.zeros((n, h, w), dtype=torch.uint8, device="cuda"), None, None) for d in dense]
        for layer in (eager, replayed):
            layer.init(dense)
            layer.step(fixed)                                  # (also the first launch of every kernel)
        ctx.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = replayed.step(fixed)
        for t, frame in enumerate(frames):
            for f, d in zip(fixed, frame):
                f.data.copy_(torch.from_numpy(d.data))
                f.mask.copy_(torch.from_numpy(d.mask))
            graph.replay()
            want = eager.step([_upload(d) for d in frame])
            ctx.sync()
            mask = to_np(want.mask)
            assert np.array_equal(to_np(out.mask), mask), f"replay {t}: mask"
            assert np.array_equal(to_np(out.data)[mask == 1], to_np(want.data)[mask == 1]), f"replay {t}: delta"
            for which in (0, 1):
                assert np.array_equal(to_np(replayed.state_tensor(which)), to_np(eager.state_tensor(which))), f"replay {t}: buffer {which}"


def _off_alignment(delta):
    """The same update with its mask 8 bytes off a 16-byte border: such a layer takes a list from memory."""
    room = torch.zeros(delta.mask.numel() + 16, dtype=torch.uint8, device="cuda")
    mask = room[8:8 + delta.mask.numel()].view(delta.mask.shape)
    mask.copy_(delta.mask)
    return pkg.Delta(delta.data, mask, delta.idx, delta.count)


@pytest.mark.parametrize("S,kind,k,stride,cin,cout,act", [
    ("f16", "conv", 3, 1, 64, 64, "relu"), ("f16", "conv", 1, 2, 48, 32, "relu6"), ("f16", "conv", 3, 2, 256, 128, "relu"),
    ("f16", "conv", 3, 1, 256, 512, "none"), ("f16", "conv", 1, 2, 512, 1032, "none"), ("f16", "conv", 3, 1, 128, 128, "none"),
    ("f32", "conv", 5, 1, 12, 20, "relu"), ("f32", "conv", 7, 2, 8, 16, "none"), ("f16", "conv", 3, 1, 20, 27, "relu"),
    ("f16", "residual", 3, 1, 64, 64, "relu"), ("f16", "projection", 1, 1, 64, 256, "relu"), ("f16", "projection", 3, 2, 64, 64, "relu"),
    ("f16", "dwconv", 3, 1, 96, 96, "relu6"), ("f32", "dwconv", 3, 2, 200, 200, "relu"), ("f16", "dwconv", 2, 2, 32, 32, "none"),
    ("f16", "add", 1, 1, 64, 64, "relu"), ("f16", "add", 1, 1, 1024, 1024, "relu"), ("f32", "add", 1, 1, 1024, 1024, "none"), ("f32", "add", 1, 1, 20, 20, "none"),
    ("f16", "upsample", 2, 1, 40, 40, "none"), ("f32", "upsample", 4, 1, 6, 6, "none"),
])
@pytest.mark.parametrize("nhw", [(1, 5, 13), (3, 12, 14), (1, 40, 51)])
def test_lists_built_in_the_kernel_and_stored_ones_give_the_same_bits(S, kind, k, stride, cin, cout, act, nhw):
    """Every kind of layer that can build its list, on maps that end 1, 24 and 24 pixels into a word of flags (and other places
    after a stride), against the same layer on a list in memory; the second layer changes between the two."""
    n, h, w = nhw
    rng = np.random.default_rng(cin + cout + h)
    dt = NP_DTYPE[S]
    code = {"conv": pkg.CONV, "residual": pkg.CONV, "projection": pkg.CONV, "strided projection": pkg.CONV, "dwconv": pkg.DWCONV, "add": pkg.ACT, "upsample": pkg.UPSAMPLE}[kind]
    pad = 0 if kind == "dwconv" and k == 2 else k // 2
    oh, ow = (h * k, w * k) if kind == "upsample" else ((h + 2 * pad - k) // stride + 1, (w + 2 * pad - k) // stride + 1)
    ins = [(n, h, w, cin)]
    proj = None
    if kind == "residual":
        ins.append((n, oh, ow, cout))
    elif kind == "add":
        ins.append(ins[0])
    elif kind in ("projection", "strided projection"):
        ps = 2 if kind == "strided projection" else stride
        proj = (24, (oh - 1) * ps + 1, (ow - 1) * ps + 1, ps)
        ins.append((n, proj[1], proj[2], 24))
    desc = pkg.make_desc(code, DT[S], n, h, w, cin, k=1 if kind == "upsample" else k, stride=stride, pad=0 if kind == "upsample" else pad, cout=cout,
                         act=pkg.ACT_CODES[act], eps=0.3, n_in=len(ins), factor=k if kind == "upsample" else 1, want_idx=0, proj=proj)
    wgt = None
    if code == pkg.CONV:
        parts = [rng.standard_normal((k, k, cin, cout)).reshape(-1) * np.sqrt(2.0 / (k * k * cin))]
        if proj:
            parts.append(rng.standard_normal(24 * cout) * np.sqrt(2.0 / 24))
        wgt = torch.from_numpy(np.concatenate(parts).astype(dt)).cuda()
    elif code == pkg.DWCONV:
        wgt = torch.from_numpy((rng.standard_normal((k, k, cin)) * 0.5).astype(dt)).cuda()
    ctx = pkg.Context(max(a * b * c for a, b, c, _ in ins + [(n, oh, ow, cout)]))
    inside, stored = (pkg.Layer(ctx, desc, wgt) for _ in range(2))
    dense = [torch.from_numpy(rng.standard_normal(shape).astype(dt)).cuda() for shape in ins]
    for layer in (inside, stored):
        layer.init(dense)
    for t, dens in enumerate((0.05, 1.0, 0.4, 0.0, 0.02, 0.9)):
        deltas = [_upload(_rand_delta(rng, shape, dens if i == 0 else dens * 0.7, S, 0.4)) for i, shape in enumerate(ins)]
        a = inside.step(deltas)
        b = stored.step([_off_alignment(d) for d in deltas] if t != 2 else deltas)
        ctx.sync()
        mask = to_np(b.mask)
        assert np.array_equal(to_np(a.mask), mask), f"step {t}: mask"
        assert np.array_equal(to_np(a.data)[mask == 1], to_np(b.data)[mask == 1]), f"step {t}: values"
        assert (a.count is None) == (b.count is None)
        if a.count is not None:
            flat = np.flatnonzero(mask.reshape(-1))
            for view in (a, b):
                assert int(to_np(view.count)[0]) == flat.size and np.array_equal(to_np(view.idx)[:flat.size], flat), f"step {t}: list"
        for which in ((0, 1) if act != "none" else ()):
            assert np.array_equal(to_np(inside.state_tensor(which)), to_np(stored.state_tensor(which))), f"step {t}: buffer {which}"
        sa, sb = inside.stats(), stored.stats()
        assert all(sa[key] == sb[key] for key in ("pixels_in", "pixels_in2", "pixels_work", "pixels_out")), f"step {t}: statistics"


@pytest.mark.parametrize("k,stride", [(1, 1), (3, 1), (3, 2), (1, 2), (7, 2)])
@pytest.mark.parametrize("at", [4, 8])
def test_mask_compact_of_unaligned_masks(k, stride, at):
    """Masks that do not start on a 16-byte border go through the two passes."""
    rng = np.random.default_rng(k + at)
    mask = (rng.random((2, 45, 67)) < 0.05).astype(np.uint8)
    want = orc.window_mask(mask, k, stride, k // 2)
    mask_b = (rng.random(want.shape) < 0.02).astype(np.uint8)
    want = want | mask_b
    views = []
    for m in (mask, mask_b):
        room = torch.zeros(m.size + 32, dtype=torch.uint8, device="cuda")
        v = room[at:at + m.size].view(m.shape)
        v.copy_(torch.from_numpy(m))
        views.append(v)
    ctx = pkg.Context(mask.size)
    got, idx, count = ctx.mask_compact(views[0], k, stride, k // 2, views[1])
    ctx.sync()
    assert np.array_equal(to_np(got), want)
    flat = np.flatnonzero(want.reshape(-1))
    assert int(to_np(count)[0]) == flat.size and np.array_equal(to_np(idx)[:flat.size], flat)


@pytest.mark.parametrize("S,k,cin,cout,res", [("f16", 1, 16, 32, False), ("f16", 3, 16, 128, True), ("f32", 1, 16, 64, False)])
@pytest.mark.parametrize("tiles", [1, 256, 257, 511, 513, 769, 1100])
def test_tiles_of_short_lists_over_the_whole_chip(S, k, cin, cout, res, tiles):
    """Lists of a tile or two per compute unit and of one more or less (the last one ends inside a tile): a workgroup takes one
    tile per round, two, three, or as many as it has room for, and every entry is worked on once."""
    n, h, w = 2, 136, 132
    rng = np.random.default_rng(tiles + cout)
    dt, eps = NP_DTYPE[S], 0.3
    ctx, layer, rconv = _conv_layers(S, k, 1, k // 2, cin, cout, (n, h, w), rng, act=pkg.ACT_RELU, eps=eps, n_in=2 if res else 1)
    radd, ract = orc.Add(S), orc.ActTrunc("relu", eps, S)
    x0 = rng.normal(0, 1, (n, h, w, cin)).astype(dt)
    s0 = rng.normal(0, 1, (n, h, w, cout)).astype(dt)
    y0 = rconv.init(x0)
    ract.init(radd.init(y0, s0) if res else y0)
    layer.init([torch.from_numpy(a).cuda() for a in ([x0, s0] if res else [x0])])
    layer.state_tensor(0).copy_(torch.from_numpy(ract.xA).cuda())
    d = _rand_delta(rng, (n, h, w, cin), 0.0, S, 0.5)
    if k == 1:
        d.mask.reshape(-1)[rng.permutation(n * h * w)[:32 * tiles - 5]] = 1
    else:                                                      # whole rows: (rows + 2) * w outputs are listed
        rows = max(1, (32 * tiles) // w - 2)
        d.mask.reshape(n * h, w)[:min(rows, h - 1)] = 1
        d.mask.reshape(n * h, w)[h + 1:h + 1 + max(0, rows - h - 1)] = 1
    d = ODelta(np.where(d.mask[..., None] == 1, rng.normal(0, 0.5, d.data.shape), np.nan).astype(dt), d.mask)
    mid = rconv.step(d).poisoned()
    sl = sum_slack(rconv, d.zero_filled()) + ulp(mid.data, S)
    ins = [_upload(d)]
    if res:
        ds = _rand_delta(rng, (n, h, w, cout), 0.001, S, 0.5)
        mid = radd.step(mid, ds).poisoned()
        sl = sl + ulp(mid.data, S)
        ins.append(_upload(ds))
    want = ract.step(mid).poisoned()
    out = layer.step(ins)
    ctx.sync()
    check_delta(out, want, S, f"{tiles} tiles", allow_mask_diff=_near_tie(ract, eps, sl), slack=sl)
    agree = to_np(out.mask) == want.mask
    for which, ref in ((0, ract.xA), (1, ract.xT)):
        assert rel_err(to_np(layer.state_tensor(which))[agree], ref[agree], slack=sl[agree]) <= TOL[S]


@pytest.mark.parametrize("S,kind,k,stride,cin,cout,act,nhw", [
    # one block of 32 pixels per workgroup, and one more than there are workgroups (blocks of 8, several each)
    ("f16", "conv", 3, 1, 32, 32, "relu", (1, 88, 90)), ("f16", "conv", 3, 1, 32, 32, "relu", (1, 91, 91)),
    # the largest map of each kind, ends inside a block and inside a word of flags
    ("f16", "residual", 3, 1, 32, 32, "relu", (5, 113, 115)), ("f16", "conv", 3, 2, 32, 32, "relu6", (4, 127, 129)), ("f32", "projection", 1, 2, 32, 32, "relu", (4, 61, 63)),
    ("f16", "add", 1, 1, 16, 16, "relu", (4, 127, 129)), ("f32", "add", 1, 1, 12, 12, "none", (2, 181, 181)), ("f16", "dwconv", 3, 1, 16, 16, "relu6", (4, 127, 129)),
    ("f16", "strided projection", 1, 1, 16, 32, "relu", (3, 127, 129)), ("f16", "strided projection", 3, 1, 32, 16, "relu", (3, 91, 91)),
    ("f16", "dwconv", 3, 2, 24, 24, "none", (4, 127, 128)), ("f16", "add", 1, 1, 512, 512, "relu", (1, 127, 129)), ("f16", "upsample", 2, 1, 16, 16, "none", (1, 63, 65)),
    # streamed weights and units: the largest outputs, and inputs beyond those that list themselves
    ("f16", "conv", 3, 2, 128, 128, "relu", (4, 127, 127)), ("f16", "conv", 1, 2, 256, 512, "none", (2, 127, 127)), ("f16", "conv", 1, 1, 384, 96, "none", (3, 45, 47)),
])
def test_blocks_of_larger_maps_give_the_bits_of_a_stored_list(S, kind, k, stride, cin, cout, act, nhw):
    """The same comparison where a workgroup compacts several blocks of pixels, up to the largest maps that take that way."""
    test_lists_built_in_the_kernel_and_stored_ones_give_the_same_bits(S, kind, k, stride, cin, cout, act, nhw)


@pytest.mark.parametrize("S,k,stride,cin,cout,act", [("f16", 3, 1, 256, 256, "none"), ("f16", 3, 1, 128, 512, "none"), ("f16", 1, 2, 256, 1040, "none"), ("f16", 3, 1, 256, 256, "relu")])
@pytest.mark.parametrize("nhw", [(1, 15, 17), (1, 16, 16), (1, 1, 257), (2, 16, 24), (8, 32, 32)])
def test_runs_of_pixels_give_the_bits_of_a_stored_list(S, k, stride, cin, cout, act, nhw):
    """The same comparison for kernels whose workgroups share runs of 256 pixels: a pixel less and more than a run, runs that list a
    part of a tile, a few tiles and all of them, one workgroup for each tile of a run and one for several."""
    test_lists_built_in_the_kernel_and_stored_ones_give_the_same_bits(S, "conv", k, stride, cin, cout, act, nhw)


@pytest.mark.parametrize("S,k,cin,cout,hw,act,residue", [("f16", 1, 64, 64, (40, 51), "relu", 0), ("f32", 3, 32, 32, (23, 29), "relu6", 1),
                                                         ("f16", 3, 128, 64, (9, 7), "relu", 0), ("f16", 1, 32, 24, (33, 65), "relu", 1),
                                                         # 64 MB of x^T and more: cleared by row
                                                         ("f16", 1, 16, 256, (257, 257), "relu", 0), ("f32", 3, 16, 64, (363, 363), "relu6", 1)])
def test_second_first_frame_clears_every_truncated_row(S, k, cin, cout, hw, act, residue):
    """A first frame after sparse steps (some of which leave values in x^T) gives the state of a layer that never saw them: the rows
    that hold values are cleared, and the steps behind it are the same."""
    rng = np.random.default_rng(cin + cout)
    dt, n, (h, w) = NP_DTYPE[S], 2, hw
    desc = pkg.make_desc(pkg.CONV, DT[S], n, h, w, cin, k=k, stride=1, pad=k // 2, cout=cout, act=pkg.ACT_CODES[act], eps=0.6, want_idx=0, xT_residue=residue)
    wgt = torch.from_numpy((rng.standard_normal((k, k, cin, cout)) * np.sqrt(2.0 / (k * k * cin))).astype(dt)).cuda()
    ctx = pkg.Context(n * h * w)
    used, fresh, looked_at = (pkg.Layer(ctx, desc, wgt) for _ in range(3))
    first, again = (torch.from_numpy(rng.standard_normal((n, h, w, cin)).astype(dt)).cuda() for _ in range(2))
    deltas = [_upload(_rand_delta(rng, (n, h, w, cin), dens, S, 0.2)) for dens in (0.3, 0.05, 0.6, 0.2)]
    for layer in (used, looked_at):
        layer.init([first])
        for d in deltas[:2]:
            layer.step([d])
    assert torch.count_nonzero(looked_at.state_tensor(1)) > 0
    looked_at.state_tensor(1).fill_(1.0)                       # whoever has the buffer may write it
    dense = [layer.init([again]) for layer in (used, fresh, looked_at)]
    assert all(torch.equal(y, dense[1]) for y in dense) or dense[0] is None
    for d in deltas[2:]:
        views = [layer.step([d]) for layer in (used, fresh, looked_at)]
        ctx.sync()
        mask = to_np(views[1].mask)
        for v in views:
            assert np.array_equal(to_np(v.mask), mask) and np.array_equal(to_np(v.data)[mask == 1], to_np(views[1].data)[mask == 1])
    used.init([first])
    ctx.sync()
    assert torch.count_nonzero(used.state_tensor(1)) == 0


@pytest.mark.parametrize("S,k,stride,cin,cout,nhw", [
    # pixels narrower than a vector whose resident weights leave less than 2 KB of LDS
    ("f16", 1, 1, 4, 3904, (1, 6, 7)), ("f16", 1, 1, 7, 3336, (1, 5, 5)), ("f32", 1, 1, 3, 3872, (1, 6, 7)), ("f32", 1, 1, 2, 1800, (2, 5, 9)),
    # narrow pixels and a window too large for one flat K dimension
    ("f16", 7, 1, 7, 40, (1, 15, 15)), ("f16", 7, 2, 6, 19, (2, 13, 11)),
    # odd channel counts above a vector: rows end inside one, at every place in it
    ("f16", 3, 1, 13, 19, (1, 14, 15)), ("f16", 1, 1, 9, 40, (2, 9, 8)), ("f16", 5, 2, 18, 24, (1, 16, 17)), ("f16", 3, 1, 43, 64, (1, 9, 30)),
    ("f16", 3, 2, 92, 16, (1, 21, 20)), ("f32", 3, 1, 7, 12, (1, 17, 16)), ("f32", 1, 1, 5, 33, (1, 12, 11)), ("f32", 7, 1, 6, 8, (1, 11, 13)),
])
def test_conv_on_rows_that_are_no_whole_vectors(S, k, stride, cin, cout, nhw):
    """The gathers of the plain kernel: value by value (with and without a flat K dimension) and one load at the row's own alignment."""
    test_conv_linear(S, k, stride, k // 2, cin, cout, nhw)


def test_first_frames_into_a_graph_leave_nothing_to_rely_on():
    """A first frame on 64 MB of x^T or more skips the rows that hold zeros already.  One that is recorded has not run: neither a
    later first frame nor its own replays may take the rows to be zero because of it."""
    rng = np.random.default_rng(3)
    n, h, w, cin, cout = 2, 257, 257, 16, 256
    desc = pkg.make_desc(pkg.CONV, DT["f16"], n, h, w, cin, k=1, cout=cout, act=pkg.ACT_RELU, eps=0.6, want_idx=0)
    wgt = torch.from_numpy(rng.standard_normal((1, 1, cin, cout)).astype(np.float16)).cuda()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = pkg.Context(n * h * w)
        twin, layer = (pkg.Layer(ctx, desc, wgt) for _ in range(2))
        at = twin.state_tensor(1).data_ptr() - twin.state.data_ptr()
        x_t = layer.state[at:at + n * h * w * cout * 2]
        x_t.fill_(0x3c)                                            # memory as it comes
        frame = torch.from_numpy(rng.standard_normal((n, h, w, cin)).astype(np.float16)).cuda()
        out = torch.empty((n, h, w, cout), dtype=torch.float16, device="cuda")
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            layer.init([frame], out)
        layer.init([frame], out)
        stream.synchronize()
        assert torch.count_nonzero(x_t) == 0, "first frame behind a recorded one"
        again = torch.cuda.CUDAGraph()
        with torch.cuda.graph(again, stream=stream):
            layer.init([frame], out)
        for g in (graph, again):
            layer.state_tensor(1).fill_(1.0)                       # whoever has the buffer may write it
            stream.synchronize()
            g.replay()
            stream.synchronize()
            assert torch.count_nonzero(x_t) == 0, "replayed first frame"
