"""GPU front end on whole frames (shape_frame_detect / _offsets / _cut)
against the FP64 oracle: brightest pixel, growth-curve r50, the 6 r50 box and
the cut-out pixels."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shape():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_0571_amd as shape
    return shape


def _gpu_detect(shape, pix, max_side=128, scale=None):
    import torch
    fr = shape.DeviceFrames(pixels=torch.from_numpy(np.ascontiguousarray(pix)).cuda(),
                            scale=None if scale is None else torch.from_numpy(scale).cuda())
    d = shape.frame_detect(fr, max_side)
    torch.cuda.synchronize()
    return fr, {k: v.cpu().numpy() for k, v in d.items()}


def _compare(pix_f64, g, max_side=128):
    """Every frame: peak, status and box exact (a box may differ only where
    6 r50 sits within 1e-6 of a rounding boundary); sky, r50 and F close."""
    ambiguous = 0
    for i in range(pix_f64.shape[0]):
        r = oracle.frame_detect(pix_f64[i], max_side)
        assert int(g["status"][i]) == r["status"], i
        assert tuple(g["peak"][i]) == r["peak"], i
        if r["status"] & oracle.NONFINITE_INPUT:
            assert tuple(g["box"][i]) == (0, 0, 0)
            assert np.isnan(g["info"][i]).all()
            continue
        sky, r50, F = (float(v) for v in g["info"][i])
        assert sky == pytest.approx(r["sky"], rel=1e-6, abs=1e-6)
        assert r50 == pytest.approx(r["r50"], rel=1e-6)
        assert F == pytest.approx(r["flux"], rel=1e-6, abs=1e-3)
        x = 6.0 * r["r50"]
        if abs(x - np.floor(x) - 0.5) < 1e-6:
            ambiguous += 1
            continue
        assert tuple(g["box"][i]) == r["box"], (i, tuple(g["box"][i]), r["box"], r["r50"])
    return ambiguous


def test_detect_and_cut_vs_oracle(shape):
    import torch
    f = synth.make_frames(48)
    fr, g = _gpu_detect(shape, f.pixels)
    assert _compare(f.pixels.astype(np.float64), g) == 0
    box = torch.from_numpy(g["box"]).cuda()
    db = shape.frame_cut(fr, box, torch.from_numpy(f.sigma).cuda())
    torch.cuda.synchronize()
    off = db.offsets.cpu().numpy()
    sides = db.sides.cpu().numpy()
    stamps = db.pixels.cpu().numpy()
    np.testing.assert_array_equal(sides, g["box"][:, 2])
    assert off[0] == 0
    np.testing.assert_array_equal(off[1:], np.cumsum(sides.astype(np.int64) ** 2)[:-1])
    for i in range(f.n):
        s = int(sides[i])
        ref = oracle.frame_cut(f.pixels[i], tuple(g["box"][i]))
        np.testing.assert_array_equal(stamps[off[i]:off[i] + s * s].reshape(s, s), ref)


def test_detect_is_deterministic(shape):
    f = synth.make_frames(16)
    _, a = _gpu_detect(shape, f.pixels)
    _, b = _gpu_detect(shape, f.pixels)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k])


def _edge_frames(H, W, rng):
    """Point sources, sources near every edge and corner, flat frames, a
    non-finite frame and a frame with no positive flux."""
    y, x = np.mgrid[0:H, 0:W]
    out = []
    for (cx, cy, s) in [(0, 0, 0.0), (W - 1, H - 1, 0.0), (W // 2, H // 2, 0.0), (3, H - 4, 2.0),
                        (W - 5, 2, 1.5), (W // 3, H // 2, 4.0), (W - 2, H // 2, 3.0)]:
        if s == 0.0:
            img = np.zeros((H, W))
            img[cy, cx] = 7.0
        else:
            img = 100.0 * np.exp(-((x - cx) ** 2 + (y - cy) ** 2) / (2 * s * s))
        out.append(img + 3.0 + rng.normal(0, 0.01, (H, W)))
    img = np.full((H, W), 2.0)
    out.append(img)                                  # flat: F = 0
    img = rng.normal(0, 1.0, (H, W))
    img[H // 2, W // 3] = np.nan
    out.append(img)                                  # non-finite
    img = -np.ones((H, W))
    img[0, :] = 50.0
    img[H // 2, W // 2] = 1.0
    out.append(img)                                  # F < 0
    img = np.zeros((H, W))
    img[1, 1] = img[H - 2, W - 2] = 5.0
    out.append(img)                                  # tie: first index wins
    return np.stack(out).astype(np.float32)


@pytest.mark.parametrize("H,W,max_side", [(37, 300, 128), (4, 4, 128), (130, 129, 32),
                                          (512, 64, 128)])
def test_edge_frames(shape, H, W, max_side):
    rng = np.random.default_rng(H * 1000 + W)
    pix = _edge_frames(H, W, rng)
    _, g = _gpu_detect(shape, pix, max_side)
    _compare(pix.astype(np.float64), g, max_side)


def test_f16_frames(shape):
    """FP16 frames with a power-of-two scale: the oracle sees the dequantised values."""
    f = synth.make_frames(8)
    peak = np.abs(f.pixels).reshape(f.n, -1).max(1)
    scale = np.exp2(np.ceil(np.log2(peak / 32768.0))).astype(np.float32)
    q = (f.pixels / scale[:, None, None]).astype(np.float16)
    _, g = _gpu_detect(shape, q, scale=scale)
    deq = q.astype(np.float64) * scale[:, None, None].astype(np.float64)
    _compare(deq, g)


def test_frames_to_fitted_objects(shape):
    """Cut-outs feed the per-object pipeline: fit parity on them as on stamps."""
    import torch
    from parity_util import check_fit, fit_parity
    f = synth.make_frames(32)
    fr, g = _gpu_detect(shape, f.pixels)
    db = shape.frame_cut(fr, torch.from_numpy(g["box"]).cuda(), torch.from_numpy(f.sigma).cuda())
    out = shape.pipeline(db, want_perr=True)
    torch.cuda.synchronize()
    pix = db.pixels.cpu().numpy()
    b = synth.Batch("frames", pix, db.offsets.cpu().numpy(), db.sides.cpu().numpy(), f.sigma,
                    np.zeros(f.n, np.uint8), f.truth, None)
    ref = oracle.pipeline(b, oracle.opts())
    gpu = {k: v.cpu().numpy() for k, v in out.items() if hasattr(v, "cpu")}
    st, failures = fit_parity(gpu, ref, b, 0xFF, "frames")
    print(st)
    r = {"fit_" + k: v for k, v in st.items()}
    r.update(n=st["n"], fit_failures=failures)
    check_fit(r, 0.8)


def _one_group_per_frame(shape, fr, max_side=128):
    """shape_frame_detect (no scratch memory)."""
    import ctypes as C

    import torch
    n, dev = fr.n, fr.device
    out = dict(info=torch.empty(n, 3, device=dev),
               peak=torch.empty(n, 2, dtype=torch.int32, device=dev),
               box=torch.empty(n, 3, dtype=torch.int32, device=dev),
               status=torch.empty(n, dtype=torch.int32, device=dev))
    f = fr.c_struct()
    rc = shape.lib.shape_frame_detect(C.byref(f), max_side, *(t.data_ptr() for t in out.values()),
                                      None)
    assert rc == shape.OK
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


# Frame sizes around the split of a frame over workgroups: one chunk (a frame
# below one batch of vectors), a frame of exactly one batch, several chunks
# with a ragged last one, frames whose starts are not 16-byte aligned (odd
# pixel counts), rows longer and much shorter than a chunk.
@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("H,W", [(4, 5), (64, 64), (64, 128), (91, 93), (517, 333), (4096, 9),
                                 (7, 4095)])
def test_split_frames_match_one_workgroup_per_frame(shape, H, W, f16):
    import torch
    rng = np.random.default_rng(H * 5000 + W)
    n = 6
    pix = rng.normal(10.0, 1.0, (n, H, W)).astype(np.float32)
    i, j = rng.integers(0, H, n), rng.integers(0, W, n)
    pix[np.arange(n), i, j] += 100.0 + 20.0 * H * W ** 0.5
    pix[1, -1, -1] = pix[1, 0, 0] = pix[1].max() + 64.0     # a tie, first and last pixel
    pix[2, H - 1, W - 1] = np.nan
    pix[3, 0, 0] = -np.inf
    pix[4] = 0.25                                           # flat: F = 0
    pix[5] -= pix[5].max()
    pix[5, H // 2, 0] = 0.0                                 # peak on the border
    scale = None
    if f16:
        scale = np.array([16.0, 16.0, 32.0, 16.0, 0.125, 16.0], np.float32)
        pix = (pix / scale[:, None, None]).astype(np.float16)
    fr, g = _gpu_detect(shape, pix, scale=scale)
    ref = _one_group_per_frame(shape, fr)
    torch.cuda.synchronize()
    for k in ("peak", "box", "status"):
        np.testing.assert_array_equal(g[k], ref[k], err_msg=k)
    # the same FP64 sums in another order, stored in FP32: the last bit, and
    # for F the rounding of sums of H W terms of size max |I|
    np.testing.assert_allclose(g["info"][:, :2], ref["info"][:, :2], rtol=2.0 ** -22)
    top = np.nan_to_num(np.abs(pix.astype(np.float64)).reshape(n, -1).max(1), posinf=0.0)
    top *= scale if f16 else 1.0
    ok = np.isfinite(ref["info"][:, 2])
    assert (np.isfinite(g["info"][:, 2]) == ok).all()
    tol = 2.0 ** -22 * np.abs(ref["info"][:, 2]) + 2.0 ** -50 * H * W * top
    assert (np.abs(g["info"][:, 2] - ref["info"][:, 2])[ok] <= tol[ok]).all()


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("H,W", [(4, 4), (64, 64), (91, 93), (192, 192)])
def test_small_frames_are_read_by_one_workgroup_each(shape, H, W, f16):
    """Frames of up to SHAPE_FRAME_WHOLE pixels give shape_frame_detect's results
    bit for bit, with and without scratch memory; pixels whose sum cancels, so
    that another order of summation would show in F."""
    import ctypes as C

    import torch
    rng = np.random.default_rng(H * W)
    n, half = 40, H * W // 2
    a = np.exp2(rng.uniform(-24, 15, (n, half)) if f16 else rng.uniform(-20, 20, (n, half)))
    v = np.concatenate([a, -a, np.zeros((n, H * W - 2 * half))], 1)
    v = rng.permuted(v, axis=1).reshape(n, H, W).astype(np.float16 if f16 else np.float32)
    fr, g = _gpu_detect(shape, v, scale=np.full(n, 0.3, np.float32) if f16 else None)
    ref = _one_group_per_frame(shape, fr)
    f, nb = fr.c_struct(), C.c_size_t()
    assert shape.lib.shape_frame_workspace_bytes(C.byref(f), C.byref(nb)) == shape.OK
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    out = {k: torch.empty(v.shape, dtype=getattr(torch, str(v.dtype)), device="cuda")
           for k, v in ref.items()}
    rc = shape.lib.shape_frame_detect_ws(C.byref(f), 128, *(t.data_ptr() for t in out.values()),
                                         ws.data_ptr(), nb.value, None)
    assert rc == shape.OK
    torch.cuda.synchronize()
    for k in ref:
        np.testing.assert_array_equal(g[k], ref[k], err_msg=k)
        np.testing.assert_array_equal(out[k].cpu().numpy(), ref[k], err_msg=k)


# Equal maxima by the pixel (in FP32 batches of 4,096 and chunks of 8,192 pixels; in
# FP16 8,192 and 32,768): in one vector, in two batches of one thread, in a chunk's
# ragged last batch, in the next chunk, in records 256 apart (which one thread of the
# combining workgroup holds), and in the last pixels.
@pytest.mark.parametrize("H,W,f16", [(1531, 1401, False), (2999, 2903, True), (517, 333, False),
                                     (517, 333, True)])
def test_first_of_equal_maxima_in_split_frames(shape, H, W, f16):
    rng = np.random.default_rng(H)
    npix, batch, chunk = H * W, 8192 if f16 else 4096, 32768 if f16 else 8192
    parts = -(-npix // chunk)
    chunk = -(-(-(-npix // parts)) // batch) * batch
    assert (-(-npix // chunk) > 256) == (H > 1000)
    last = (npix - 1) // chunk * chunk
    sets = [[1000, 1001], [5 + 4 * 7, 5 + 4 * 7 + batch], [batch - 1, batch], [chunk - 1, chunk],
            [chunk + 9, 2 * chunk + 1, 9 + batch], [last - 1, last, npix - 1], [npix - 2, npix - 1],
            [W, npix // 2]]
    if H > 1000:
        sets += [[3 + chunk, 3 + 257 * chunk], [257 * chunk, 2 * chunk], [0, chunk, 256 * chunk]]
    pix = rng.normal(10.0, 1.0, (len(sets), npix)).astype(np.float16 if f16 else np.float32)
    for k, at in enumerate(sets):
        pix[k, at] = 900.0
    fr, g = _gpu_detect(shape, pix.reshape(-1, H, W), scale=np.ones(len(sets), np.float32) if f16 else None)
    ref = _one_group_per_frame(shape, fr)
    first = np.array([min(at) for at in sets])
    np.testing.assert_array_equal(g["peak"], np.stack([first % W, first // W], 1))
    for k in ("peak", "box", "status"):
        np.testing.assert_array_equal(g[k], ref[k], err_msg=k)
    # sky: an FP64 mean in another order; F: sums of H W terms of at most 900
    np.testing.assert_allclose(g["info"][:, 0], ref["info"][:, 0], rtol=2.0 ** -22)
    assert (np.abs(g["info"][:, 2] - ref["info"][:, 2])
            <= 2.0 ** -22 * np.abs(ref["info"][:, 2]) + 2.0 ** -50 * npix * 900.0).all()
