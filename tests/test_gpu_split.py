"""Split conv tiles (shapes 12 .. 19: both operands as three bf16 parts, six
products summed in fp32) at the sizes where they can go wrong: channel tails,
tiles that cross rows and images, strides, windows of one row or column,
padded 1 x 1 windows, merged destinations, an input ReLU, and values outside
the range in which the parts are exact (a second run of the tile, in fp32).

Tolerance: an operand's three parts add up to it; with |x2| <= 2^-8 and |x3| <=
2^-17 of x's power of two the products left out (x2 w3, x3 w2, x3 w3) are below
2^-24 + 2^-34 of a product, and the fp32 sums of n terms err by at most n 2^-24
of the sum of the terms' magnitudes; per output the error is at most (K + 8)
2^-24 sum |x| |w|, K the reduction length (the six products of 16 terms are
K 6 / 16 additions, so K >= 1 leaves room for the products left out)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
I = pytest.importorskip("paper_2011_01302_amd")
from oracle import evaluator as E          # noqa: E402

DEV = "cuda:0"
SPLIT = list(range(12, 20))


def conv_op(name, cout, k, pad, stride=1, pre=0, post=0):
    return {"name": name, "kind": "conv", "in": ["x"], "cout": cout, "kh": k[0], "kw": k[1], "sh": stride,
            "sw": stride, "ph": pad[0], "pw": pad[1], "pre_relu": pre, "post_relu": post}


def graph(monkeypatch, batch, c, h, w, ops, ten):
    monkeypatch.setenv("IOS_CONV_TILE", "1")          # no tile measurement at set-up
    g = I.Graph({"batch": batch, "inputs": [{"name": "x", "c": c, "h": h, "w": w}], "ops": ops,
                 "outputs": [o["name"] for o in ops]}, ten)
    return g


def launch(g, stages, strategies, x, ops, h, w):
    q = I.ios_schedule_from_stages(g.handle, stages, strategies)
    d = torch.from_numpy(x).to(DEV)
    outs = []
    for o in ops:
        ho, wo = (h + 2 * o["ph"] - o["kh"]) // o["sh"] + 1, (w + 2 * o["pw"] - o["kw"]) // o["sw"] + 1
        outs.append(torch.full((g.batch, o["cout"], ho, wo), float("nan"), device=DEV))
    for _ in range(2):
        I.ios_run(g.handle, q, [d.data_ptr()], [t.data_ptr() for t in outs], 0)
    torch.cuda.synchronize()
    assert I.ios_device_status(g.handle) == 0
    I.ios_schedule_destroy(q)
    return [t.cpu().numpy().astype(np.float64) for t in outs]


def reference(x, wt, b, o):
    """(exact, bound) of one conv."""
    s, p = (o["sh"], o["sw"]), (o["ph"], o["pw"])
    ref = E.conv2d(x, wt, b, s, p, o["pre_relu"], o["post_relu"])
    xa = np.maximum(x, 0) if o["pre_relu"] else np.abs(x)
    mag = E.conv2d(xa, np.abs(wt), np.abs(b), s, p)
    return ref, (wt[0].size + 8) * 2.0 ** -24 * mag


CASES = {
    # batch, c, h, w, cout, window, pad, stride, input ReLU
    "tails": (3, 5, 7, 9, 33, (3, 3), (1, 1), 1, 0),
    "one channel past a chunk": (2, 17, 11, 6, 70, (5, 5), (2, 2), 1, 0),
    "stride over images": (4, 33, 8, 8, 40, (3, 3), (1, 1), 2, 0),
    "stride past the window": (2, 24, 9, 7, 31, (2, 2), (0, 0), 3, 0),
    "gather, stride 2": (2, 24, 9, 5, 31, (1, 1), (0, 0), 2, 0),
    "gather, padded": (2, 16, 5, 5, 32, (1, 1), (1, 1), 1, 0),
    "column window": (3, 20, 6, 6, 65, (7, 1), (3, 0), 1, 0),
    "row window": (1, 64, 17, 17, 96, (1, 7), (0, 3), 1, 0),
    "several rounds": (1, 200, 33, 20, 64, (3, 3), (1, 1), 1, 0),
    "many chunks, one pixel": (1, 530, 1, 1, 130, (1, 1), (0, 0), 1, 0),
    "input ReLU": (2, 20, 9, 9, 40, (3, 3), (1, 1), 1, 1),
    "tile edge": (1, 16, 16, 16, 128, (3, 3), (1, 1), 1, 0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_split_shapes(name, monkeypatch):
    n, c, h, w, cout, k, pad, stride, pre = CASES[name]
    rng = np.random.default_rng(len(name) * 1000 + c)
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    wt = (rng.standard_normal((cout, c) + k) * (2.0 / (c * k[0] * k[1])) ** 0.5).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    ops = [conv_op("a", cout, k, pad, stride, pre)]
    g = graph(monkeypatch, n, c, h, w, ops, {"a.w": wt, "a.b": b})
    ref, bound = reference(x, wt, b, ops[0])
    for t in SPLIT:
        I.ios_set_conv_tile(g.handle, g.tid["a"], t)
        got, = launch(g, [[g.tid["a"]]], [I.IOS_CONCURRENT], x, ops, h, w)
        assert np.all(np.abs(got - ref) <= bound), (name, t, float((np.abs(got - ref) / bound).max()))
    g.close()


@pytest.mark.parametrize("tile", [12, 15, 17, 19])
def test_split_merge_has_every_destination(tile, monkeypatch):
    """A 1x1 and a 3x3 conv of one input as one merge stage (two routes), and
    the same pair as one concurrent stage."""
    rng = np.random.default_rng(7)
    x = rng.standard_normal((2, 19, 10, 13)).astype(np.float32)
    ops = [conv_op("a", 37, (1, 1), (0, 0), post=1), conv_op("b", 50, (3, 3), (1, 1), post=1)]
    ten = {}
    for o in ops:
        ten[o["name"] + ".w"] = (rng.standard_normal((o["cout"], 19, o["kh"], o["kw"])) * 0.2).astype(np.float32)
        ten[o["name"] + ".b"] = rng.standard_normal(o["cout"]).astype(np.float32)
    g = graph(monkeypatch, 2, 19, 10, 13, ops, ten)
    u = [g.tid["a"], g.tid["b"]]
    monkeypatch.setenv("IOS_CONV_TILE", str(tile))
    for i in u:
        I.ios_set_conv_tile(g.handle, i, tile)
    for stages, strat in (([u], [I.IOS_MERGE]), ([u], [I.IOS_CONCURRENT])):
        got = launch(g, stages, strat, x, ops, 10, 13)
        for o, y in zip(ops, got):
            ref, bound = reference(x, ten[o["name"] + ".w"], ten[o["name"] + ".b"], o)
            bound = bound * (9 * 19 + 8) / (19 * o["kh"] * o["kw"] + 8)     # merged: the larger window's length
            assert np.all(np.abs(y - ref) <= bound), (tile, strat, o["name"])
    g.close()


@pytest.mark.parametrize("scale", [1e-38, 1e-30, 1e-14, 1e25, 1e30, "inf", "nan"])
def test_split_values_out_of_range(scale, monkeypatch):
    """Inputs so small or large that bf16 parts would lose bits or overflow,
    an infinity and a NaN: as plain fp32 sums give them (1e-30, 1e-14: in range)."""
    rng = np.random.default_rng(3)
    n, c, h, w, cout = 2, 20, 9, 9, 40
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    if scale == "inf":
        x[1, 7, 4, 4] = np.inf
    elif scale == "nan":
        x[0, 3, 0, 8] = np.nan
    else:
        x = (x * np.float32(scale)).astype(np.float32)
    wt = (rng.standard_normal((cout, c, 3, 3)) * 0.1).astype(np.float32)
    b = np.zeros(cout, np.float32)
    ops = [conv_op("a", cout, (3, 3), (1, 1))]
    g = graph(monkeypatch, n, c, h, w, ops, {"a.w": wt, "a.b": b})
    ref, bound = reference(x, wt, b, ops[0])
    fine = np.isfinite(ref)
    for t in SPLIT:
        I.ios_set_conv_tile(g.handle, g.tid["a"], t)
        got, = launch(g, [[g.tid["a"]]], [I.IOS_CONCURRENT], x, ops, h, w)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), (scale, t)
        assert np.array_equal(got[~fine & ~np.isnan(ref)], ref[~fine & ~np.isnan(ref)]), (scale, t)
        # 1e-38: products fall below the normal numbers, whose spacing is 2^-149
        assert np.all(np.abs(got - ref)[fine] <= bound[fine] + c * 9 * 2.0 ** -149), (scale, t)
    g.close()


def profiled(g, ids, strategy, tiles):
    """Stage times with the first unit on each of the tile shapes."""
    out = []
    for t in tiles:
        I.ios_set_conv_tile(g.handle, ids[0], t)
        out.append(I.ios_profile_stage(g.handle, ids, strategy, 5, 20, 5))
    return out


def test_split_beside_sepconv(monkeypatch):
    """A large conv on a split shape beside SEPCONVs of each kind of tile: right,
    and that shape runs (16 x 32, shape 1, takes more than twice its time)."""
    rng = np.random.default_rng(23)
    n, c, h, w = 16, 96, 35, 36
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    ops = [conv_op("a", 96, (3, 3), (1, 1)),
           {"name": "s", "kind": "sepconv", "in": ["x"], "cout": 40, "kh": 3, "kw": 3, "sh": 1, "sw": 1, "ph": 1,
            "pw": 1, "pre_relu": 1, "post_relu": 0}]
    ten = {"a.w": (rng.standard_normal((96, c, 3, 3)) / 30).astype(np.float32),
           "a.b": rng.standard_normal(96).astype(np.float32),
           "s.dw": (rng.standard_normal((c, 1, 3, 3)) / 3).astype(np.float32),
           "s.pw": (rng.standard_normal((40, c, 1, 1)) / 10).astype(np.float32),
           "s.b": rng.standard_normal(40).astype(np.float32)}
    monkeypatch.setenv("IOS_SEP_TILE", "0")
    g = graph(monkeypatch, n, c, h, w, ops, ten)
    u = [g.tid["a"], g.tid["s"]]
    ref, bound = reference(x, ten["a.w"], ten["a.b"], ops[0])
    r = np.maximum(x, 0).astype(np.float64)
    sref = E.conv2d(E.depthwise(r, ten["s.dw"], (1, 1)), ten["s.pw"], ten["s.b"])
    mag = E.conv2d(E.depthwise(r, np.abs(ten["s.dw"]), (1, 1)), np.abs(ten["s.pw"]), np.abs(ten["s.b"]))
    for sep in (0, 3, 7):
        I.ios_set_unit_tiling(g.handle, u[1], sep, -1)
        for t in (13, 17):
            I.ios_set_conv_tile(g.handle, u[0], t)
            y, z = launch(g, [u], [I.IOS_CONCURRENT], x, ops, h, w)
            assert np.all(np.abs(y - ref) <= bound), (sep, t)
            assert np.all(np.abs(z - sref) <= (c + 18) * 2.0 ** -24 * mag), (sep, t)
    I.ios_set_unit_tiling(g.handle, u[1], 7, -1)
    split, small = profiled(g, u, I.IOS_CONCURRENT, (14, 1))
    assert split < 0.75 * small, (split, small)
    g.close()


def test_split_that_the_merged_window_does_not_admit(monkeypatch):
    """A 1 x 1 conv on a split shape merged with a 5 x 5 one whose input rows do
    not fit: the stage runs on the conv's best other shape, not on 16 x 32 (251
    and 294 us; two runs of one shape differ by about 1%)."""
    rng = np.random.default_rng(29)
    ops = [conv_op("a", 512, (1, 1), (0, 0)), conv_op("b", 16, (5, 5), (2, 2))]
    ten = {}
    for o in ops:
        ten[o["name"] + ".w"] = (rng.standard_normal((o["cout"], 64, o["kh"], o["kw"])) / 30).astype(np.float32)
        ten[o["name"] + ".b"] = rng.standard_normal(o["cout"]).astype(np.float32)
    monkeypatch.delenv("IOS_CONV_TILE", raising=False)  # (the other shape is a measured one)
    g = I.Graph({"batch": 1, "inputs": [{"name": "x", "c": 64, "h": 40, "w": 310}], "ops": ops, "outputs": ["a", "b"]}, ten)
    u = [g.tid["a"], g.tid["b"]]
    split, small = profiled(g, u, I.IOS_MERGE, (14, 1))
    assert split < 0.93 * small, (split, small)
    x = rng.standard_normal((1, 64, 40, 310)).astype(np.float32)
    I.ios_set_conv_tile(g.handle, u[0], 14)
    for o, y in zip(ops, launch(g, [u], [I.IOS_MERGE], x, ops, 40, 310)):
        ref, bound = reference(x, ten[o["name"] + ".w"], ten[o["name"] + ".b"], o)
        bound = bound * (25 * 64 + 8) / (64 * o["kh"] * o["kw"] + 8)
        assert np.all(np.abs(y - ref) <= bound), o["name"]
    g.close()


def mixed(rng, shape, scale):
    """Ordinary values, the first rows of the first image scaled: tiles that
    hold both, and windows that hold the scaled ones only."""
    x = rng.standard_normal(shape).astype(np.float32)
    x[0, :, :5] *= np.float32(scale)
    return x


@pytest.mark.parametrize("scale", [1e-31, 1e-36, 1e-40, 1e22])
def test_split_mixed_magnitudes(scale, monkeypatch):
    """A region of tiny (or huge) values beside ordinary ones in one tile: its
    outputs keep the bound of their own terms, a few steps of 2^-149 apart (six
    products a term, each rounded there)."""
    rng = np.random.default_rng(11)
    x = mixed(rng, (2, 20, 9, 9), scale)
    wt = (rng.standard_normal((40, 20, 3, 3)) * 0.1).astype(np.float32)
    wt[3, 5] = 0
    b = np.zeros(40, np.float32)
    ops = [conv_op("a", 40, (3, 3), (1, 1))]
    g = graph(monkeypatch, 2, 20, 9, 9, ops, {"a.w": wt, "a.b": b})
    ref, bound = reference(x, wt, b, ops[0])
    bound = bound + 6 * 180 * 2.0 ** -149
    for t in SPLIT:
        I.ios_set_conv_tile(g.handle, g.tid["a"], t)
        got, = launch(g, [[g.tid["a"]]], [I.IOS_CONCURRENT], x, ops, 9, 9)
        assert np.all(np.abs(got - ref) <= bound), (scale, t, float((np.abs(got - ref) / bound).max()))
    g.close()


@pytest.mark.parametrize("scale", [1e-36, 1e24, "inf"])
def test_split_merge_values_out_of_range(scale, monkeypatch):
    """The fp32 path of a merge stage with two destinations."""
    rng = np.random.default_rng(19)
    x = mixed(rng, (2, 19, 10, 13), 1.0 if scale == "inf" else scale)
    if scale == "inf":
        x[1, 7, 6, 4] = np.inf
    ops = [conv_op("a", 37, (1, 1), (0, 0), post=1), conv_op("b", 50, (3, 3), (1, 1), post=1)]
    ten = {}
    for o in ops:
        ten[o["name"] + ".w"] = (rng.standard_normal((o["cout"], 19, o["kh"], o["kw"])) * 0.2).astype(np.float32)
        ten[o["name"] + ".b"] = np.zeros(o["cout"], np.float32)
    g = graph(monkeypatch, 2, 19, 10, 13, ops, ten)
    u = [g.tid["a"], g.tid["b"]]
    for tile in SPLIT:
        monkeypatch.setenv("IOS_CONV_TILE", str(tile))
        got = launch(g, [u], [I.IOS_MERGE], x, ops, 10, 13)
        for o, y in zip(ops, got):
            # the merged conv is the 3 x 3 window of both: an infinity beside a 1 x 1 window meets its zero taps
            w3 = np.zeros((o["cout"], 19, 3, 3), np.float32)
            w3[:, :, (3 - o["kh"]) // 2:(3 + o["kh"]) // 2, (3 - o["kw"]) // 2:(3 + o["kw"]) // 2] = ten[o["name"] + ".w"]
            o3 = conv_op(o["name"], o["cout"], (3, 3), (1, 1))
            with np.errstate(invalid="ignore"):
                ref, bound = reference(x, w3, ten[o["name"] + ".b"], o3)
            if o["post_relu"]:
                ref = np.fmax(ref, 0)                    # the kernels' ReLU takes a NaN to 0
            fine = np.isfinite(ref)
            assert np.array_equal(np.isnan(y), np.isnan(ref)), (tile, o["name"])
            assert np.array_equal(y[~fine & ~np.isnan(ref)], ref[~fine & ~np.isnan(ref)]), (tile, o["name"])
            # (no bound where a NaN became 0: the values are the same there)
            bound = np.where(np.isnan(bound), 0, bound) + 6 * 171 * 2.0 ** -149
            with np.errstate(invalid="ignore"):
                assert np.all((np.abs(y - ref) <= bound)[fine]), (tile, o["name"])
    g.close()


SEP_CASES = {
    # batch, c, h, w, cout, window: rows odd and even, tiles within and across images, tails, several channel groups
    "even rows, last tile short": (1, 20, 6, 42, 40, 5),
    "odd rows": (2, 17, 11, 13, 70, 3),
    "tiles across images": (5, 33, 5, 6, 31, 5),
    "one row per image": (3, 16, 1, 8, 32, 3),
    "more than 192 channels": (1, 40, 8, 12, 400, 3),
    "rows of four": (2, 18, 9, 4, 33, 5),
    "rows of three (the staged tile)": (2, 18, 9, 3, 33, 3),
    "odd pixel count": (1, 48, 13, 13, 64, 5),
}


@pytest.mark.parametrize("name", list(SEP_CASES))
def test_sep_split(name, monkeypatch):
    """SEPCONV choices 7 and 8.  A depthwise value errs by at most (k k + 1)
    2^-24 of its terms' magnitudes, the pointwise sum as a conv's."""
    n, c, h, w, cout, k = SEP_CASES[name]
    rng = np.random.default_rng(c * 100 + k)
    x = rng.standard_normal((n, c, h, w)).astype(np.float32)
    dw = (rng.standard_normal((c, 1, k, k)) / k).astype(np.float32)
    pw = (rng.standard_normal((cout, c, 1, 1)) / c ** 0.5).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    check_sep(monkeypatch, x, dw, pw, b, k)


@pytest.mark.parametrize("scale", [1e-38, 1e-20, 1e25, "inf", "nan"])
def test_sep_split_values_out_of_range(scale, monkeypatch):
    rng = np.random.default_rng(5)
    x = rng.standard_normal((2, 20, 9, 10)).astype(np.float32)
    if scale == "inf":
        x[1, 7, 4, 4] = np.inf
    elif scale == "nan":
        x[0, 3, 0, 8] = np.nan          # the input ReLU takes a NaN to 0
    else:
        x = (x * np.float32(scale)).astype(np.float32)
    dw = (rng.standard_normal((20, 1, 3, 3)) / 3).astype(np.float32)
    pw = (rng.standard_normal((33, 20, 1, 1)) / 5).astype(np.float32)
    check_sep(monkeypatch, x, dw, pw, np.zeros(33, np.float32), 3)


@pytest.mark.parametrize("scale", [1e-31, 1e-36, 1e22])
def test_sep_split_mixed_magnitudes(scale, monkeypatch):
    rng = np.random.default_rng(13)
    x = mixed(rng, (2, 20, 9, 10), scale)
    dw = (rng.standard_normal((20, 1, 3, 3)) / 3).astype(np.float32)
    pw = (rng.standard_normal((33, 20, 1, 1)) / 5).astype(np.float32)
    check_sep(monkeypatch, x, dw, pw, np.zeros(33, np.float32), 3)


def test_sep_split_tiny_output_channel(monkeypatch):
    """Pointwise weights out of the parts' range: another tile runs the choice."""
    rng = np.random.default_rng(17)
    x = rng.standard_normal((1, 20, 9, 10)).astype(np.float32)
    dw = (rng.standard_normal((20, 1, 3, 3)) / 3).astype(np.float32)
    pw = (rng.standard_normal((33, 20, 1, 1)) / 5).astype(np.float32)
    pw[4] *= np.float32(1e-36)
    check_sep(monkeypatch, x, dw, pw, np.zeros(33, np.float32), 3)


def check_sep(monkeypatch, x, dw, pw, b, k):
    n, c, h, w = x.shape
    cout = pw.shape[0]
    op = {"name": "a", "kind": "sepconv", "in": ["x"], "cout": cout, "kh": k, "kw": k, "sh": 1, "sw": 1, "ph": k // 2,
          "pw": k // 2, "pre_relu": 1, "post_relu": 0}
    monkeypatch.setenv("IOS_SEP_TILE", "0")
    g = graph(monkeypatch, n, c, h, w, [op], {"a.dw": dw, "a.pw": pw, "a.b": b})
    r = np.where(np.isnan(x), 0, np.maximum(x, 0)).astype(np.float64)
    d = E.depthwise(r, dw, (k // 2, k // 2))
    da = E.depthwise(np.where(np.isinf(r), 0, r), np.abs(dw), (k // 2, k // 2))
    with np.errstate(invalid="ignore"):
        ref = E.conv2d(d, pw, b)
    bound = (c + k * k + 9) * 2.0 ** -24 * E.conv2d(da, np.abs(pw), np.abs(b)) + c * k * k * 2.0 ** -149
    fine = np.isfinite(ref)
    for t in (7, 8)[:1 if 2 * w > 64 else 2]:          # choice 8 holds two rows in 64 pixels
        I.ios_set_unit_tiling(g.handle, g.tid["a"], t, -1)
        got, = launch(g, [[g.tid["a"]]], [I.IOS_CONCURRENT], x, [op], h, w)
        assert np.array_equal(np.isnan(got), np.isnan(ref)), t
        assert np.array_equal(got[~fine & ~np.isnan(ref)], ref[~fine & ~np.isnan(ref)]), t
        assert np.all(np.abs(got - ref)[fine] <= bound[fine]), (t, float((np.abs(got - ref)[fine] / bound[fine]).max()))
    g.close()


def test_split_refused_for_weights_out_of_range():
    """Weights that are not finite, above 2^40 or all below 2^-30, and one below
    2^-110 among ordinary ones: no split shape."""
    for v in (np.inf, np.nan, 2.0 ** 41, 2.0 ** -31, 2.0 ** -111):
        wt = np.full((8, 16, 3, 3), v, np.float32)
        if v == 2.0 ** -111:
            wt[:7] = 0.5
        g = I.Graph({"batch": 1, "inputs": [{"name": "x", "c": 16, "h": 5, "w": 5}],
                     "ops": [conv_op("a", 8, (3, 3), (1, 1))], "outputs": ["a"]},
                    {"a.w": wt, "a.b": np.zeros(8, np.float32)})
        for t in SPLIT:
            with pytest.raises(I.IosError):
                I.ios_set_conv_tile(g.handle, g.tid["a"], t)
        g.close()
