"""The matrix kernel on bf16 pieces (SCONV_VARIANT=piece): every geometry at the edges of its tiles, whole and split
along the channels, from every form of the filters; integer inputs exact, the others within the parity bar and as close
to the 64-bit sums as an fp32 sum of the same length; non-finite and tiny values as the fp32 kernels treat them."""
import re

import numpy as np
import pytest
import torch

import conftest
import oracle
import workloads
import paper_1909_09927_amd as sconv
from parity import check_forward, check_pool_forward, to_dev

pytestmark = pytest.mark.gpu

# (geometry, (N, C, H, W, K, R, S, stride, pad, groups, pool), split "whole tiles,1,slices" or None)
CASES = [
    ("a128x128", (1, 16, 11, 12, 128, 3, 3, 1, 1, 1, None), None),        # one chunk; the last tile four windows long
    ("a128x128", (2, 48, 19, 23, 70, 3, 3, 1, 1, 1, None), "3,1,2"),      # ragged filter block, whole tiles and split ones
    ("a128x64", (5, 33, 7, 7, 129, 3, 3, 1, 1, 1, None), "0,1,3"),        # ragged channels, one filter in the last block
    ("a128x64", (2, 32, 9, 57, 64, 3, 3, 1, 0, 1, None), None),           # several column strips, the last one narrower
    ("a64x128", (2, 96, 14, 14, 96, 3, 3, 1, 1, 3, None), None),          # grouped, half a filter block
    ("a64x128", (4, 64, 3, 5, 40, 3, 3, 1, 2, 1, None), "0,1,2"),         # padding wider than a tile's share of the map
    ("s128x64", (2, 33, 19, 23, 70, 3, 3, 2, 1, 1, None), None),          # stride 2
    ("s128x64", (3, 20, 14, 14, 96, 3, 3, 3, 0, 1, None), None),          # stride 3, no padding
    ("b64x128", (2, 96, 14, 14, 96, 3, 3, 1, 1, 3, None), None),          # as a64x128 and p128x64, small products apart
    ("b64x128", (2, 48, 19, 23, 70, 3, 3, 1, 1, 1, None), "3,1,2"),
    ("u128x64", (2, 48, 13, 15, 130, 3, 3, 1, 1, 1, (2, 2, 2)), "3,1,2"),
    ("u128x64", (1, 16, 12, 9, 64, 3, 3, 1, 1, 1, (2, 2, 1)), None),
    ("p128x128", (2, 32, 14, 14, 128, 3, 3, 1, 1, 1, (2, 2, 2)), None),
    ("p128x64", (2, 48, 13, 15, 130, 3, 3, 1, 1, 1, (2, 2, 2)), "3,1,2"),
    ("p128x64", (1, 16, 12, 9, 64, 3, 3, 1, 1, 1, (2, 2, 1)), None),      # overlapping pooling windows
    ("p128x64", (1, 16, 14, 15, 64, 3, 3, 1, 1, 1, (2, 2, 3)), None),     # pooling windows with gaps
    ("p128x64", (1, 20, 13, 12, 70, 3, 3, 1, 0, 1, (2, 2, 4)), None),
    ("c128x64", (2, 100, 15, 14, 96, 1, 1, 1, 0, 1, None), "1,1,2"),      # 1x1, ragged channels, strips across images
    ("c128x64", (1, 64, 7, 7, 96, 1, 1, 2, 0, 2, None), None),            # 1x1, stride 2 (a tile's positions fit on small maps only), grouped
    ("c128x64", (2, 35, 9, 7, 129, 1, 1, 1, 0, 1, None), None),           # filters of 35 channels: read one by one, the last block one filter
    ("c128x64", (1, 146, 15, 14, 258, 1, 1, 1, 0, 2, None), "1,1,2"),
    ("c128x64", (1, 20, 9, 7, 129, 1, 1, 1, 0, 1, None), None),           # whole fragments past the last channel
    ("q128x64", (2, 256, 14, 16, 96, 1, 1, 1, 0, 1, (2, 2, 2)), None),
    ("q128x64", (3, 70, 6, 9, 129, 1, 1, 1, 0, 1, (2, 2, 2)), "2,1,2"),   # ragged channels, one filter in the last block, an odd column left out
    ("q128x64", (1, 35, 5, 40, 64, 1, 1, 1, 0, 1, (2, 2, 2)), None),      # strips
    # taps dealt to the wavefronts
    ("t3x64", (1, 33, 7, 7, 33, 3, 3, 1, 1, 1, None), None),              # one channel in the second chunk, one filter in the second block
    ("t3x64", (2, 128, 9, 13, 40, 3, 3, 2, 1, 2, None), "1,1,2"),
    ("t5x64", (3, 16, 7, 7, 32, 5, 5, 1, 2, 1, None), None),              # one chunk, the last tile 19 windows long
    ("t5x64", (1, 3, 13, 11, 20, 5, 5, 2, 0, 1, None), None),             # fewer channels than half a lane's eight, stride 2, no padding
    ("t5x64", (1, 3, 33, 29, 20, 5, 5, 1, 0, 1, None), None),
    ("t5x64", (2, 50, 8, 12, 70, 5, 5, 1, 2, 2, None), "2,1,2"),
    ("t5x128", (2, 40, 12, 31, 33, 5, 5, 1, 2, 1, None), "0,1,3"),
    ("t7x64", (1, 24, 13, 6, 33, 7, 7, 1, 3, 1, None), None),
    ("t7x96", (1, 17, 13, 14, 31, 7, 7, 2, 3, 1, None), "0,1,2"),         # stride 2
    ("t7x96", (2, 17, 21, 18, 33, 7, 7, 1, 3, 1, None), "5,1,2"),
    ("tp5x128", (2, 48, 13, 15, 33, 5, 5, 1, 2, 1, (2, 2, 2)), "1,1,3"),
    ("tp5x128", (1, 16, 11, 9, 32, 5, 5, 1, 0, 1, (2, 2, 1)), None),
    ("tp5x128", (1, 20, 17, 11, 40, 5, 5, 1, 2, 1, (2, 2, 4)), None),
    ("tp7x96", (1, 20, 14, 14, 40, 7, 7, 1, 3, 1, (2, 2, 2)), None),
]


def _pin(monkeypatch, geom, split, src):
    monkeypatch.setenv("SCONV_VARIANT", "piece")
    monkeypatch.setenv("SCONV_PIECE_GEOM", geom)
    for name, value in (("SCONV_PIECE_SPLIT", split), ("SCONV_PIECE_SRC", src)):
        if value is None:
            monkeypatch.delenv(name, raising=False)
        else:
            monkeypatch.setenv(name, value)


def _assert_it_runs(desc, pool, ws, geom, split, src):
    """The pinned geometry, split and form of the filters have a plan (without one the window-row kernel would run)."""
    name = sconv.sconv_launch_name(desc, pool is not None, ws.numel() if ws is not None else 0)
    want = f"piece/model:{geom}/{('pieces', 'prepared', 'stored')[int(src)]}"
    if split is None:
        assert name == want or name.startswith(want + "/")
    else:
        whole, _, slices = split.split(",")
        assert name.startswith(f"{want}/{whole}+") and name.endswith(f"x{slices}")


@pytest.mark.parametrize("src", ["0", "1", "2"])     # pieces in the workspace, prepared filters, filters as stored
@pytest.mark.parametrize("geom,shp,split", CASES)
def test_geometries_splits_and_filter_sources(device, monkeypatch, geom, shp, split, src):
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    prep = src == "1"
    if prep and (R != 3 or stride != 1 or pad != 1 or (C // groups) % 16 or pool and pool != (2, 2, 2)):
        pytest.skip("no prepared layout for this layer")
    if geom[0] == "t" and src != "2":
        pytest.skip("reads the filters as stored")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    for integer in (False, True):
        layer, x, w = workloads.make_random_case(400, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6, integer)
        xd, wd = to_dev(x), to_dev(w)
        bias = to_dev(np.arange(K, dtype=np.float32) % 7 - 3) if prep else None
        _pin(monkeypatch, geom, split, src)
        _assert_it_runs(sconv.desc_for(xd, wd, stride, pad, groups, pool, True, None, prep), pool, ws, geom, split, src)
        wp = sconv.sconv_filter_prep(wd, groups, stride, pad) if prep else None
        kw = dict(ws=ws, bias=bias, wprep=wp) if prep else dict(ws=ws)
        if pool:
            got = sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, **kw)
        else:
            got = sconv.sconv_forward(xd, wd, stride, pad, groups, **kw)
        torch.cuda.synchronize()
        got = got.cpu().numpy().astype(np.float64)
        ref, scale = oracle.conv(x, w, stride, pad, groups, relu=False)
        if prep:
            b = bias.cpu().numpy().astype(np.float64)[None, :, None, None]
            ref, scale = ref + b, scale + np.abs(b)
        if pool:
            p = torch.nn.functional.max_pool2d
            ref = p(torch.from_numpy(np.maximum(ref, 0.0)), pool[:2], pool[2]).numpy()
            scale = p(torch.from_numpy(scale), pool[:2], pool[2]).numpy()
        assert got.shape == ref.shape
        if integer:
            assert np.array_equal(got, ref)
        else:
            # fp32 accumulation of L terms in any order stays within L * 2^-24 of the scale; the six products of three
            # pieces leave out 3 * 2^-24 of a term's size
            bound = (C // groups * R * S + 3) * 2.0 ** -24
            assert (np.abs(got - ref) <= bound * scale).all()
            assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)   # measured 1e-7 to 2e-7


@pytest.mark.parametrize("geom,src", [("a128x64", "2"), ("a128x128", "0"), ("a64x128", "1"), ("t3x64", "2")])
def test_values_outside_the_pieces_range(device, monkeypatch, geom, src):
    """Inf, NaN, values that overflow when rounded to bf16 and values whose pieces fall below bf16's range give what the
    window-row kernel gives; zeros of the map are skipped (0 * Inf adds nothing)."""
    _, x, w = workloads.make_random_case(401, 2, 32, 14, 14, 70, 3, 3, 1, 1, 1, None, 0.6)
    x_bad = x.copy()
    x_bad[0, 3, 5, 5], x_bad[1, 7, 2, 3], x_bad[1, 9, 9, 9] = np.inf, np.nan, 3.4e38
    w_bad = w.copy()
    w_bad[5, 4, 1, 1], w_bad[66, 0, 0, 0] = np.inf, -np.inf
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    for xi, wi in ((x_bad, w), (x, w_bad), (x * np.float32(1e-36), w), (x, w * np.float32(1e-38))):
        xd, wd = to_dev(xi), to_dev(wi)
        _pin(monkeypatch, geom, None, src)
        _assert_it_runs(sconv.desc_for(xd, wd, 1, 1, 1, None, True, None, src == "1"), None, ws, geom, None, src)
        wp = sconv.sconv_filter_prep(wd) if src == "1" else None
        y = sconv.sconv_forward(xd, wd, 1, 1, ws=ws, wprep=wp).cpu().numpy()
        monkeypatch.setenv("SCONV_VARIANT", "rows")
        r = sconv.sconv_forward(xd, wd, 1, 1, ws=ws).cpu().numpy()
        assert np.array_equal(np.isnan(y), np.isnan(r)) and np.array_equal(np.isinf(y), np.isinf(r))
        ok = np.isfinite(r)
        _, scale = oracle.conv(np.where(np.isfinite(xi), xi, 0), np.where(np.isfinite(wi), wi, 0), 1, 1, 1)
        assert (np.abs(y[ok].astype(np.float64) - r[ok]) <= 1e-4 * scale[ok]).all()


@pytest.mark.parametrize("xe,we", [(-134, 0), (-124, 50), (-120, 45), (-140, 70), (0, -134), (45, -126), (-60, -60), (90, -60), (105, -70), (-70, 105),
                                   (-14, -118)])
@pytest.mark.parametrize("geom,src,shp", [
    ("a128x64", "2", (2, 32, 14, 14, 70, 3, 3, 1, 1, 1, None)), ("a128x128", "0", (2, 32, 14, 14, 70, 3, 3, 1, 1, 1, None)),
    ("a64x128", "1", (2, 32, 14, 14, 70, 3, 3, 1, 1, 1, None)), ("c128x64", "0", (2, 100, 15, 14, 96, 1, 1, 1, 0, 1, None)),
    ("c128x64", "2", (2, 100, 15, 14, 96, 1, 1, 1, 0, 1, None)), ("p128x64", "0", (2, 32, 14, 14, 70, 3, 3, 1, 1, 1, (2, 2, 2))),
    ("t3x64", "2", (2, 32, 14, 14, 70, 3, 3, 1, 1, 1, None)), ("tp5x128", "2", (1, 20, 14, 14, 40, 5, 5, 1, 2, 1, (2, 2, 2))),
])
def test_operands_of_any_size(device, monkeypatch, geom, src, shp, xe, we):
    """Maps and filters scaled by powers of two down into fp32's subnormals (a few bits left: the operands are what the call is
    given) and up to where the pieces overflow: as close to the 64-bit sums as ordinary operands are."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(403, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6)
    x, w = np.ldexp(x, xe), np.ldexp(w, we)
    xd, wd = to_dev(x), to_dev(w)
    _pin(monkeypatch, geom, None, src)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    _assert_it_runs(sconv.desc_for(xd, wd, stride, pad, groups, pool, True, None, src == "1"), pool, ws, geom, None, src)
    kw = dict(ws=ws, wprep=sconv.sconv_filter_prep(wd)) if src == "1" else dict(ws=ws)
    got = (sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, **kw) if pool else sconv.sconv_forward(xd, wd, stride, pad, groups, **kw))
    got = got.cpu().numpy().astype(np.float64)
    ref, scale = oracle.conv(x, w, stride, pad, groups, relu=False)
    if pool:
        p = torch.nn.functional.max_pool2d
        ref = p(torch.from_numpy(np.maximum(ref, 0.0)), pool[:2], pool[2]).numpy()
        scale = p(torch.from_numpy(scale), pool[:2], pool[2]).numpy()
    # the bound of the test above; results and partial sums below fp32's range round to multiples of 2^-149
    bound = (C // groups * R * S + 3) * 2.0 ** -24
    assert np.isfinite(got).all() and (np.abs(got - ref) <= bound * scale + 4 * 2.0 ** -149).all()
    if np.median(scale) > 2.0 ** -120:
        assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("shp", [
    (8, 64, 28, 28, 96, 3, 3, 1, 1, 1, None), (2, 256, 14, 14, 256, 3, 3, 1, 1, 1, (2, 2, 2)), (8, 128, 14, 14, 256, 1, 1, 1, 0, 1, None),
    (8, 64, 28, 28, 64, 3, 3, 2, 1, 1, None), (4, 40, 33, 31, 60, 3, 3, 1, 0, 2, None),
])
def test_default_plans(device, monkeypatch, shp):
    """The decomposition the model picks - with the lent workspace, without one, and the same result on every call."""
    monkeypatch.setenv("SCONV_VARIANT", "piece")
    layer, x, w = workloads.make_random_case(402, *shp[:10], shp[10], 0.7)
    (check_pool_forward if layer.pool else check_forward)(layer, x, w)
    xd, wd = to_dev(x), to_dev(w)
    call = (lambda **k: sconv.sconv_pool_forward(xd, wd, layer.pool, layer.stride, layer.pad, layer.groups, **k)) if layer.pool else \
        (lambda **k: sconv.sconv_forward(xd, wd, layer.stride, layer.pad, layer.groups, relu=True, **k))
    a, b, c = call(), call(), call(ws=None)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert np.linalg.norm((a - c).cpu().numpy()) <= 1e-6 * np.linalg.norm(c.cpu().numpy())


@pytest.mark.parametrize("shp,ws,z", [
    ((4, 128, 28, 28, 256, 3, 3, 1, 1, 1, None), False, None), ((4, 128, 28, 28, 256, 3, 3, 1, 1, 1, None), True, None),
    ((8, 64, 28, 28, 64, 3, 3, 2, 1, 1, None), True, None), ((8, 512, 14, 14, 256, 1, 1, 1, 0, 1, (2, 2, 2)), True, None),
    ((4, 256, 28, 28, 256, 3, 3, 1, 1, 1, None), True, 0.5), ((4, 256, 28, 28, 256, 3, 3, 1, 1, 1, None), True, 0.95),
    ((1, 16, 28, 28, 32, 3, 3, 1, 1, 1, None), True, None), ((4, 48, 7, 7, 128, 5, 5, 1, 2, 1, None), False, None),
])
def test_launch_name_is_what_runs(device, monkeypatch, capfd, shp, ws, z):
    """The piece kernel says on stderr what it launches (SCONV_TRACE_PLAN): that, or nothing, is what sconv_launch_name named."""
    monkeypatch.setenv("SCONV_TRACE_PLAN", "1")
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(404, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.7)
    xd, wd = to_dev(x), to_dev(w)
    d = sconv.desc_for(xd, wd, stride, pad, groups, pool, True, z)
    wsb = torch.empty(sconv.sconv_workspace_size(d, pool is not None), dtype=torch.uint8, device="cuda") if ws else None
    sconv.sconv_env_refresh()
    name = sconv.sconv_launch_name(d, pool is not None, wsb.numel() if ws else 0)
    sconv.sconv_set_workspace(None)       # ws=None would take the lent one
    try:
        capfd.readouterr()
        if pool:
            sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, ws=wsb, zero_ratio=z)
        else:
            sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=wsb, zero_ratio=z)
        torch.cuda.synchronize()
    finally:
        sconv.sconv_set_workspace(conftest._WORKSPACE)
    said = [line.split()[1] for line in capfd.readouterr().err.splitlines() if line.startswith("piece ")]
    assert said == ([name.split(":")[1].split("/")[0] + ":"] if name.startswith("piece/model:") else [])


def _off_by_one(a):
    """The array on the device, 4 bytes past a 16-byte boundary."""
    buf = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
    view = buf[1:].view(*a.shape)
    view.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    assert view.data_ptr() % 16 == 4 and view.is_contiguous()
    return view


@pytest.mark.parametrize("geom,src,shp", [
    ("a128x64", "0", (2, 33, 14, 13, 70, 3, 3, 1, 1, 1, None)), ("a128x64", "2", (2, 33, 14, 13, 70, 3, 3, 1, 1, 1, None)),
    ("p128x64", "2", (2, 33, 14, 13, 70, 3, 3, 1, 1, 1, (2, 2, 2))), ("c128x64", "2", (2, 100, 15, 14, 96, 1, 1, 1, 0, 1, None)),
    ("c128x64", "2", (2, 35, 9, 7, 129, 1, 1, 1, 0, 1, None)), ("t5x64", "2", (1, 33, 7, 7, 33, 5, 5, 1, 2, 1, None)),
])
def test_operands_off_a_16_byte_boundary(device, monkeypatch, geom, src, shp):
    """Maps, filters and results that are slices of something larger: the same bits as from aligned copies."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(405, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6)
    _pin(monkeypatch, geom, None, src)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    _assert_it_runs(sconv.desc_for(to_dev(x), to_dev(w), stride, pad, groups, pool, True), pool, ws, geom, None, src)

    def call(xd, wd, out=None):
        if pool:
            return sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, ws=ws, out=out)
        return sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=ws, out=out)
    aligned = call(to_dev(x), to_dev(w))
    out = _off_by_one(np.full(tuple(aligned.shape), -1.0, np.float32))
    call(_off_by_one(x), _off_by_one(w), out)
    torch.cuda.synchronize()
    assert torch.equal(aligned, out)


@pytest.mark.parametrize("shp,forms", [
    ((8, 64, 28, 28, 96, 3, 3, 2, 1, 1, None), ("s128x64/stored/0+25x4", "s128x64/stored")),
    ((16, 128, 56, 56, 128, 3, 3, 2, 1, 1, None), ("s128x64/pieces", "s128x64/stored")),
    ((1, 512, 7, 7, 512, 3, 3, 1, 1, 1, None), ("t3x64/stored/0+16x16", "t3x64/stored/0+16x8", "t3x64/stored")),
])
def test_workspaces_of_any_size(device, monkeypatch, shp, forms):
    """From what the plan can use down to nothing: pieces and partial sums go where they fit, the bytes behind the workspace
    stay as they are, every result within the bar."""
    monkeypatch.setenv("SCONV_VARIANT", "piece")
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(406, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6)
    xd, wd = to_dev(x), to_dev(w)
    d = sconv.desc_for(xd, wd, stride, pad, groups, pool, True)
    full = sconv.sconv_workspace_size(d)
    ref, scale = oracle.conv(x, w, stride, pad, groups, relu=True)
    names = []
    for size in (full, full // 2, full // 8, full // 64, 4096, 16):
        buf = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        names.append(sconv.sconv_launch_name(d, False, size))
        y = sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=buf[:size])
        torch.cuda.synchronize()
        assert (buf[size:] == 0xA5).all()
        assert (np.abs(y.cpu().numpy().astype(np.float64) - ref) <= 1e-4 * scale).all()
    assert {"piece/model:" + f for f in forms} <= set(names)


@pytest.mark.parametrize("geom,split,src,shp", [
    ("s128x64", "10,1,2", "0", (8, 64, 28, 28, 64, 3, 3, 2, 1, 1, None)), ("t3x64", "0,1,4", "2", (1, 256, 14, 14, 256, 3, 3, 1, 1, 1, None)),
])
def test_launches_captured_into_a_graph(device, monkeypatch, geom, split, src, shp):
    """Pieces of the filters written and split tiles added inside the graph: every replay gives what an eager call gives on the
    map and the filters as they are then."""
    _pin(monkeypatch, geom, split, src)
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(407, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6)
    xd, wd = to_dev(x), to_dev(w)
    d = sconv.desc_for(xd, wd, stride, pad, groups, pool, True)
    ws, ws2 = (torch.empty(sconv.sconv_workspace_size(d), dtype=torch.uint8, device="cuda") for _ in range(2))
    _assert_it_runs(d, None, ws, geom, split, src)
    st = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    out = sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=ws)
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        with torch.cuda.graph(graph, stream=st):
            sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=ws, out=out)
    torch.cuda.synchronize()
    for rep in range(4):
        _, xn, wn = workloads.make_random_case(408 + rep, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6)
        xd.copy_(torch.from_numpy(xn))
        wd.copy_(torch.from_numpy(wn))
        out.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, sconv.sconv_forward(xd, wd, stride, pad, groups, relu=True, ws=ws2))


@pytest.mark.parametrize("shp,call,families", [
    ((2, 512, 28, 28, 512, 3, 3, 1, 1, 1, None), "prepared", ("tap", "quad")), ((2, 256, 28, 28, 256, 3, 3, 1, 1, 1, None), "prepared", ("tap", "quad")),
    ((2, 128, 56, 56, 128, 3, 3, 2, 1, 1, None), "ws", ("wide",)), ((2, 512, 28, 28, 256, 1, 1, 1, 0, 1, None), "ws", ("quad1x1",)),
    ((8, 128, 56, 56, 128, 3, 3, 1, 1, 1, None), "ws", ("tap", "quad")), ((16, 64, 56, 56, 64, 3, 3, 1, 1, 1, None), "ws", ("tap", "quad")),
    ((4, 256, 56, 56, 256, 3, 3, 1, 1, 1, None), "ws", ("tap", "quad")), ((16, 22, 33, 33, 256, 3, 3, 1, 1, 1, None), "ws", ("gen",)),
])
@pytest.mark.parametrize("z", [0.5, 0.7])
def test_no_further_from_64_bit_sums_than_the_kernels_it_replaces(device, monkeypatch, shp, call, families, z):
    """Relative error against the oracle's 64-bit sums of the plan that the model takes: at most a twentieth above that of the other
    kernels (whose own moves by that much with the seed)."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(412, N, C, H, W, K, R, S, stride, pad, groups, pool, z)
    xd, wd = to_dev(x), to_dev(w)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    kw = dict(ws=ws, wprep=sconv.sconv_filter_prep(wd)) if call == "prepared" else dict(ws=ws)
    desc = sconv.desc_for(xd, wd, stride, pad, groups, pool, False, z, call == "prepared")
    ref, _ = oracle.conv(x, w, stride, pad, groups, relu=False)

    def error():
        y = sconv.sconv_forward(xd, wd, stride, pad, groups, zero_ratio=z, **kw).cpu().numpy().astype(np.float64)
        return np.linalg.norm(y - ref) / np.linalg.norm(ref)
    monkeypatch.delenv("SCONV_VARIANT", raising=False)
    name = sconv.sconv_launch_name(desc, False, ws.numel())
    if not name.startswith("piece/"):      # (at these small batches: the one geometry that takes over at larger ones, pinned)
        assert R == 1 or stride == 2
        geom = "c128x64" if R == 1 else "s128x64"
        _pin(monkeypatch, geom, None, "0")
        _assert_it_runs(desc, pool, ws, geom, None, "0")
    mine = error()
    for name in ("SCONV_PIECE_GEOM", "SCONV_PIECE_SRC", "SCONV_VARIANT"):
        monkeypatch.delenv(name, raising=False)
    for family in families:
        if family != "quad1x1":
            monkeypatch.setenv("SCONV_VARIANT", family)
        assert not sconv.sconv_launch_name(desc, False, ws.numel()).startswith("piece")
        other = error()
        print(f"{family}: {mine:.3e} against {other:.3e}")
        assert mine <= 1.05 * other


PAIRS = [
    ("a128x64", (1, 16, 11, 12, 128, 3, 3, 1, 1, 1, None), None),         # one chunk, the last tile four windows long
    ("a128x64", (5, 33, 7, 7, 129, 3, 3, 1, 1, 1, None), "0,1,3"),        # ragged channels, one filter in the last block, a chunk per slice
    ("a128x64", (2, 96, 9, 57, 192, 3, 3, 1, 0, 2, None), "2,1,2"),       # grouped, column strips, whole and split tiles
    ("a128x64", (1, 64, 13, 21, 40, 3, 3, 1, 2, 1, None), "0,1,2"),       # padding 2, half a filter block
    ("u128x64", (2, 48, 13, 15, 130, 3, 3, 1, 1, 1, (2, 2, 2)), "3,1,2"),
    ("u128x64", (1, 16, 12, 9, 64, 3, 3, 1, 1, 1, (2, 2, 1)), None),
]


def _pairs_call(monkeypatch, geom, split, shp, x, w, relu=False, prepared=False):
    """split "x2": blocks of two of the geometry's tiles."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    xd, wd = to_dev(x), to_dev(w)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    block = split == "x2"
    _pin(monkeypatch, geom + "x2" if block else geom, None if block else split, "3")
    kw = dict(ws=ws, wprep=sconv.sconv_filter_prep(wd, groups)) if prepared else dict(ws=ws)
    name = sconv.sconv_launch_name(sconv.desc_for(xd, wd, stride, pad, groups, pool, True, prepared=prepared), pool is not None, ws.numel())
    slices = ("/x2" if block else r"(/\d+\+\d+x\d+)?" if split is None else "" if split.endswith(",1,1") else
              r"/{}\+\d+x{}".format(*split.split(",")[::2]))
    assert re.fullmatch(f"piece/model:{geom}/{'prepared' if prepared else 'pieces'}-f16k{slices}", name), name
    y = (sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, **kw) if pool else sconv.sconv_forward(xd, wd, stride, pad, groups, relu, **kw))
    return y.cpu().numpy().astype(np.float64)


def _reference(shp, x, w):
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    ref, scale = oracle.conv(x, w, stride, pad, groups, relu=False)
    if pool:
        p = torch.nn.functional.max_pool2d
        ref = p(torch.from_numpy(np.maximum(ref, 0.0)), pool[:2], pool[2]).numpy()
        scale = p(torch.from_numpy(scale), pool[:2], pool[2]).numpy()
    return ref, scale


@pytest.mark.parametrize("geom,shp,split", PAIRS + [(geom, shp, "x2") for geom, shp, _ in PAIRS])
def test_pairs(device, monkeypatch, geom, shp, split):
    """Tile edges, remainders, splits: integers exact; the others within what fp32 sums of the same length may be off by, and within
    5e-7 in all (measured 1e-7 to 1.5e-7)."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    for integer in (False, True):
        _, x, w = workloads.make_random_case(420, N, C, H, W, K, R, S, stride, pad, groups, pool, 0.6, integer)
        got = _pairs_call(monkeypatch, geom, split, shp, x, w)
        ref, scale = _reference(shp, x, w)
        if integer:
            assert np.array_equal(got, ref)
        else:
            # as three pieces; of a pair's last bits the half ulp of either operand, and the fourth product, are left out: 2 * 2^-24 + 2^-22
            assert (np.abs(got - ref) <= (C // groups * 9 + 6) * 2.0 ** -24 * scale).all()
            assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("split", [None, "x2"])
@pytest.mark.parametrize("what", ["images", "channels up", "channels down", "late", "small among large", "subnormal", "huge", "small weights", "filters",
                                  "weight range", "inf", "nan", "inf weight"])
def test_pairs_hold_maps_and_filters_of_any_range(device, monkeypatch, what, split):
    """The scale of a pair follows the chunks; what no scale holds is summed from three pieces: as close as ever, element by element."""
    shp = (6, 64, 6, 7, 140, 3, 3, 1, 1, 1, None)
    _, x, w = workloads.make_random_case(421, *shp[:10], None, 0.6)
    rng = np.random.default_rng(5)
    if what == "images":               # several in one tile
        x = np.ldexp(x, np.array([0, -40, 20, -70, 3, 0])[:, None, None, None])
    elif what == "channels up":        # every chunk another scale
        x = np.ldexp(x, (np.arange(64) // 16 * 9)[None, :, None, None])
    elif what == "channels down":
        x = np.ldexp(x, (np.arange(64) // 16 * -25)[None, :, None, None])
    elif what == "late":               # the first chunks hold nothing
        x[:, :40] = 0
    elif what == "small among large":  # windows of values 2^-33 of their neighbours
        x[:, :, :3] = np.ldexp(x[:, :, :3], -33)
    elif what == "subnormal":
        x = np.ldexp(x, -135)
        w = np.ldexp(w, 60)
    elif what == "huge":
        x = np.ldexp(x, 110)
        w = np.ldexp(w, -70)
    elif what == "small weights":
        w = np.ldexp(w, -135)
        x = np.ldexp(x, 60)
    elif what == "filters":            # neighbouring filters 2^-60 apart
        w = np.ldexp(w, (np.arange(140) % 3 * -30)[:, None, None, None])
    elif what == "weight range":       # a filter no pair holds
        w = np.ldexp(w, np.where(rng.random(w.shape) < 0.5, -45, 0))
    elif what == "inf":
        x[2, 20, 3, 3] = np.inf
    elif what == "nan":
        x[2, 20, 3, 3] = np.nan
    else:
        w[77, 3, 1, 1] = -np.inf
    x, w = x.astype(np.float32), w.astype(np.float32)
    got = _pairs_call(monkeypatch, "a128x64", split, shp, x, w)
    bad = ~np.isfinite(_pairs_rows(monkeypatch, shp, x, w))
    xf, wf = np.where(np.isfinite(x), x, 0), np.where(np.isfinite(w), w, 0)
    ref, scale = _reference(shp, xf, wf)
    assert np.array_equal(~np.isfinite(got), bad) and bad.any() == (what in ("inf", "nan", "inf weight"))
    assert (np.abs(got - ref) <= (64 * 9 + 6) * 2.0 ** -24 * scale + 4 * 2.0 ** -149)[~bad].all()


@pytest.mark.parametrize("split", ["0,1,1", "0,1,2", "x2"])
@pytest.mark.parametrize("pool", [None, (2, 2, 2)])
@pytest.mark.parametrize("up_x,up_w", [(-62, -62), (-76, -50), (-30, -96), (-99, -27), (55, 55), (104, 54), (54, 104)])
def test_pairs_of_maps_and_filters_both_small_or_both_large(device, monkeypatch, up_x, up_w, split, pool):
    """What undoes the two scales is far outside fp32's range where the results are ordinary numbers: sums of 2^-126 and more, windows of
    zeros, and, where the large elements overflow, the windows that hold small ones against small weights."""
    shp = (6, 64, 6, 7, 140, 3, 3, 1, 1, 1, pool)
    _, x, w = workloads.make_random_case(423, *shp[:10], None, 0.6)
    x, w = np.abs(x), w.copy()
    x[2:4] = 0
    if up_x + up_w > 128:      # images 4 and 5: every second channel 2^-24 of the others' elements, against weights 2^-24 of the others
        x[4:, ::2] = 0
        x[4:] = np.ldexp(x[4:], -24)
        w[:, 1::2] = np.ldexp(w[:, 1::2], -24)
        x, w = np.where(np.abs(x) < 2.0 ** -24.5, 0, x), np.where(np.abs(w) < 2.0 ** -28, 2.0 ** -28, w)
    x, w = np.ldexp(x, up_x).astype(np.float32), np.ldexp(w, up_w).astype(np.float32)
    got = _pairs_call(monkeypatch, "u128x64" if pool else "a128x64", split, shp, x, w)
    ref, scale = _reference(shp, x, w)
    assert np.abs(ref).max() > 2.0 ** -126 and not ref[2 if pool else 3, :, 0 if pool else 3].any()
    fits = scale < 2.0 ** 126
    assert fits.all() == (up_x + up_w < 128) and fits[4:].all()
    assert (np.abs(got - ref) <= (64 * 9 + 6) * 2.0 ** -24 * scale + 4 * 2.0 ** -149)[fits].all()


@pytest.mark.parametrize("split", ["0,1,1", "0,1,2", "x2"])
@pytest.mark.parametrize("step", [40, -40, 11, -11])
def test_pairs_of_chunks_whose_scales_keep_moving(device, monkeypatch, step, split):
    """Chunks that are each 2^step of the one before: windows that hold elements of the first one only keep their sums."""
    shp = (6, 96, 6, 7, 140, 3, 3, 1, 1, 1, None)
    _, x, w = workloads.make_random_case(424, *shp[:10], None, 0.6)
    x[0, 16:] = 0
    x[3, :80] = 0
    x = np.ldexp(x, (np.arange(96) // 16 * step - 2.5 * step).astype(int)[None, :, None, None]).astype(np.float32)
    got = _pairs_call(monkeypatch, "a128x64", split, shp, x, w)
    ref, scale = _reference(shp, x, w)
    assert (np.abs(got - ref) <= (96 * 9 + 6) * 2.0 ** -24 * scale + 4 * 2.0 ** -149).all()


@pytest.mark.parametrize("split", [None, "x2"])
@pytest.mark.parametrize("spread_x,spread_w", [(0, 0), (26, 0), (0, 26), (26, 26), (0, 29), (29, 0)])
def test_pairs_hold_every_single_product(device, monkeypatch, spread_x, spread_w, split):
    """One nonzero element a window, so nothing averages: its product with any weight, over the range that pairs hold (26 octaves) and just
    past it.  A value is held to 2^-23 of itself and the product left out is 2^-22; a fp32 rounding or two of the result besides."""
    shp = (2, 32, 12, 15, 140, 3, 3, 1, 1, 1, None)
    rng = np.random.default_rng(6)
    x, w = np.zeros(shp[:4]), rng.uniform(1, 2, (140, 32, 3, 3)) * np.exp2(-rng.integers(0, spread_w + 1, (140, 32, 3, 3)))
    at = np.ix_(range(2), range(1, 12, 3), range(1, 15, 3))
    c = rng.integers(0, 32, (2, 4, 5))
    x[at[0], c, at[1], at[2]] = rng.uniform(1, 2, c.shape) * np.exp2(-rng.integers(0, spread_x + 1, c.shape))
    x, w = x.astype(np.float32), w.astype(np.float32)
    got = _pairs_call(monkeypatch, "a128x64", split, shp, x, w)
    ref, scale = _reference(shp, x, w)
    assert (scale > 0).all()
    assert (np.abs(got - ref) <= (2.0 ** -22 + 2 * 2.0 ** -23 + 2 * 2.0 ** -24) * scale).all()


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("split,pool", [("0,1,1", None), ("2,1,2", None), ("x2", None), ("0,1,1", (2, 2, 2)), ("x2", (2, 2, 2))])
@pytest.mark.parametrize("what", [0, 1, 3, 5, "every", "filter", "filters"])
def test_tiles_go_on_from_three_pieces(device, monkeypatch, what, split, pool, prepared):
    """One element that pairs do not hold, in chunk `what` (or in every one): the chunks before it from pairs, it and those after it from
    three pieces, of either form of the filters.  A filter that pairs do not hold: its whole block from pieces."""
    shp = (4, 96, 6, 7, 140, 3, 3, 1, 1, 1, pool)
    _, x, w = workloads.make_random_case(425, *shp[:10], None, 0.6)
    x, w = x.copy(), w.copy()
    if what == "filter":
        w[77, 50, 1, 1] = 1e-20
    elif what == "filters":
        w[::9, 50, 1, 1] = 1e-40
    else:
        for c in range(96) if what == "every" else (16 * what + 3,):
            x[1, c, 2, 3] = 2.0 ** -30
    got = _pairs_call(monkeypatch, "u128x64" if pool else "a128x64", split, shp, x, w, prepared=prepared)
    ref, scale = _reference(shp, x, w)
    assert (np.abs(got - ref) <= (96 * 9 + 6) * 2.0 ** -24 * scale).all()
    assert np.linalg.norm(got - ref) <= 2e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("what", ["integers", "plain", "element", "filter"])
@pytest.mark.parametrize("shp,split", [((1, 1840, 5, 5, 130, 3, 3, 1, 1, 1, None), "0,1,1"), ((1, 64, 13, 21, 40, 3, 3, 1, 2, 1, None), "0,1,2"),
                                       ((1, 1840, 5, 5, 130, 3, 3, 1, 1, 1, None), "x2"), ((1, 64, 13, 21, 40, 3, 3, 1, 2, 1, None), "x2")])
def test_pairs_without_room_for_pieces(device, monkeypatch, shp, split, what):
    """Pairs alone fill the workspace, so what they do not hold is summed from the filters as stored; 1840 channels: one filter in LDS, not two."""
    _, x, w = workloads.make_random_case(427, *shp[:10], None, 0.6, what == "integers")
    x, w = x.copy(), w.copy()
    if what == "element":
        x[0, 40, 2, 3] = 2.0 ** -30
    elif what == "filter":
        w[17, 20, 1, 1] = 1e-20
    got = _pairs_call(monkeypatch, "a128x64", split, shp, x, w)
    ref, scale = _reference(shp, x, w)
    if what == "integers":
        assert np.array_equal(got, ref)
    else:
        assert (np.abs(got - ref) <= (shp[1] * 9 + 6) * 2.0 ** -24 * scale).all()
        assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("prepared", [False, True])
@pytest.mark.parametrize("what", ["integers", "plain", "bias", "scales", "element", "filter"])
@pytest.mark.parametrize("geom,shp", [
    ("a128x64x2", (1, 16, 8, 16, 128, 3, 3, 1, 1, 1, None)),      # one tile, one chunk
    ("a128x64x2", (3, 48, 14, 13, 129, 3, 3, 1, 1, 1, None)),     # one filter in the last block, the last tile ragged, three chunks
    ("a128x64x2", (2, 96, 9, 57, 192, 3, 3, 1, 1, 2, None)),      # grouped, half a filter block, column strips
    ("a128x64x2", (1, 112, 28, 28, 40, 3, 3, 1, 1, 1, None)),     # 28 columns: as many positions as are staged
    ("u128x64x2", (2, 64, 13, 15, 130, 3, 3, 1, 1, 1, (2, 2, 2))),
])
def test_blocks(device, monkeypatch, geom, shp, what, prepared):
    """128 filters x 128 windows: edges of tiles, filters and chunks; scales that move, what pairs do not hold; within the bound of test_pairs."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(428, *shp[:10], None, 0.6, what == "integers")
    x, w = x.copy(), w.copy()
    if what == "scales":
        x = np.ldexp(x, (np.arange(C) // 16 * 11 - 33).astype(int)[None, :, None, None]).astype(np.float32)
    elif what == "element":
        x[0, C - 1, 2, 3] = 2.0 ** -30
    elif what == "filter":
        w[K // 2, 3, 1, 1] = 1e-20
    xd, wd = to_dev(x), to_dev(w)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    _pin(monkeypatch, geom, None, "3")
    name = sconv.sconv_launch_name(sconv.desc_for(xd, wd, stride, pad, groups, pool, True, prepared=prepared), pool is not None, ws.numel())
    assert name == f"piece/model:{geom[:-2]}/{'prepared' if prepared else 'pieces'}-f16k/x2"
    b = np.random.default_rng(9).normal(size=K).astype(np.float32) if what == "bias" and prepared else None
    kw = dict(ws=ws, wprep=sconv.sconv_filter_prep(wd, groups), bias=to_dev(b) if b is not None else None) if prepared else dict(ws=ws)
    got = (sconv.sconv_pool_forward(xd, wd, pool, stride, pad, groups, **kw) if pool
           else sconv.sconv_forward(xd, wd, stride, pad, groups, relu=False, **kw)).cpu().numpy().astype(np.float64)
    ref, scale = oracle.conv(x, w, stride, pad, groups, relu=False)
    if b is not None:
        ref, scale = ref + b.astype(np.float64)[None, :, None, None], scale + np.abs(b.astype(np.float64))[None, :, None, None]
    if pool:
        p = torch.nn.functional.max_pool2d
        ref = p(torch.from_numpy(np.maximum(ref, 0.0)), pool[:2], pool[2]).numpy()
        scale = p(torch.from_numpy(scale), pool[:2], pool[2]).numpy()
    if what == "integers":
        assert np.array_equal(got, ref)
    else:
        assert (np.abs(got - ref) <= (C // groups * 9 + 7) * 2.0 ** -24 * scale).all()
        assert np.linalg.norm(got - ref) <= 5e-7 * np.linalg.norm(ref)   # as in test_pairs


def _pairs_rows(monkeypatch, shp, x, w):
    """The window-row kernel, which skips zeros of the map."""
    for name in ("SCONV_PIECE_GEOM", "SCONV_PIECE_SRC", "SCONV_PIECE_SPLIT"):
        monkeypatch.delenv(name, raising=False)
    monkeypatch.setenv("SCONV_VARIANT", "rows")
    return sconv.sconv_forward(to_dev(x), to_dev(w), shp[7], shp[8], shp[9]).cpu().numpy()


@pytest.mark.parametrize("shp,z,call,three", [
    ((8, 256, 56, 56, 256, 3, 3, 1, 1, 1, None), 0.6, "ws", ("a128x64", "0")), ((8, 512, 28, 28, 512, 3, 3, 1, 1, 1, None), 0.5, "ws", ("s128x64", "0")),
    ((8, 512, 28, 28, 512, 3, 3, 1, 1, 1, None), 0.75, "prepared", ("a128x64", "1")),
    ((8, 640, 14, 14, 384, 3, 3, 1, 1, 1, None), 0.8, "ws", None), ((2, 320, 56, 56, 128, 3, 3, 1, 1, 1, None), 0.5, "ws", ("a128x128", "2")),
])
def test_pairs_are_no_further_from_64_bit_sums_than_what_they_replace(device, monkeypatch, shp, z, call, three):
    """The plan the model takes against the one it would take without pairs (three pieces, or None: the vector kernel); seeds move either by
    a twentieth."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(422, N, C, H, W, K, R, S, stride, pad, groups, pool, z)
    xd, wd = to_dev(x), to_dev(w)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    kw = dict(ws=ws, wprep=sconv.sconv_filter_prep(wd)) if call == "prepared" else dict(ws=ws)
    desc = sconv.desc_for(xd, wd, stride, pad, groups, pool, False, z, call == "prepared")
    wn = wd.double().reshape(K, -1)
    ref = torch.stack([wn @ torch.nn.functional.unfold(xd[n:n + 1].double(), 3, padding=pad)[0] for n in range(2)]).reshape(2, K, H, W)

    def error():
        y = sconv.sconv_forward(xd, wd, stride, pad, groups, zero_ratio=z, **kw)[:2].double()
        return float((y - ref).norm() / ref.norm())
    monkeypatch.delenv("SCONV_VARIANT", raising=False)
    assert "-f16" in sconv.sconv_launch_name(desc, False, ws.numel())
    mine = error()
    if three:
        _pin(monkeypatch, three[0], None, three[1])
    else:
        monkeypatch.setenv("SCONV_VARIANT", "tap")
    assert "-f16" not in sconv.sconv_launch_name(desc, False, ws.numel())
    other = error()
    print(f"{mine:.3e} against {other:.3e}")
    assert mine <= 1.05 * other


@pytest.mark.parametrize("shp,z", [((7, 262, 58, 58, 48, 3, 3, 1, 1, 1, None), 0.68), ((7, 656, 37, 27, 96, 3, 3, 1, 0, 1, None), 0.9),
                                   ((8, 661, 24, 14, 127, 3, 3, 1, 1, 1, None), 0.84)])
def test_pairs_leave_the_taps_kernel_where_it_is_closer(device, monkeypatch, shp, z):
    """Layers that the taps kernel served as fast as three pieces do: what runs now is no further from 64-bit sums; seeds move either by a
    twentieth."""
    N, C, H, W, K, R, S, stride, pad, groups, pool = shp
    _, x, w = workloads.make_random_case(426, *shp[:10], None, z)
    xd, wd = to_dev(x), to_dev(w)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    ref = (wd.double().reshape(K, -1) @ torch.nn.functional.unfold(xd[:1].double(), 3, padding=pad)[0]).reshape(1, K, H + 2 * pad - 2, -1)

    def error():
        y = sconv.sconv_forward(xd, wd, stride, pad, groups, zero_ratio=z if C == 262 else None, ws=ws)[:1].double()
        return float((y - ref).norm() / ref.norm())
    for name in ("SCONV_VARIANT", "SCONV_PIECE_GEOM", "SCONV_PIECE_SRC", "SCONV_PIECE_SPLIT"):
        monkeypatch.delenv(name, raising=False)
    mine = error()
    _pin(monkeypatch, "t3x64", None, None)
    other = error()
    print(f"{mine:.3e} against {other:.3e}")
    assert mine <= 1.05 * other
