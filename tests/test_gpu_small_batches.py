"""GPU: the kernels that small batches take give the results of the ones that
large batches take, bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shape():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_0571_amd as shape
    return shape


def _repeat(shape, db, n):
    """A batch of n stamps that are db's, over and over (the same pixels)."""
    import torch
    idx = torch.arange(n, device=db.device) % db.n
    pick = lambda t: None if t is None else t[idx].contiguous()   # noqa: E731
    return shape.DeviceBatch(pixels=db.pixels, sigma=pick(db.sigma), offsets=pick(db.offsets),
                             sides=pick(db.sides), scale=pick(db.scale), model=pick(db.model))


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_mixed_sides_one_launch_equals_launch_per_form(shape, storage):
    """Mixed sides (every form, with stamps that cannot be processed): up to
    65,536 stamps take one launch, more take a launch per form."""
    import torch
    b = synth.make("uneven", count=640, storage=storage)
    b.sides[:8] = [4, 8, 16, 63, 64, 65, 96, 97]     # both ends of every form
    db = shape.DeviceBatch.from_host(b, "cuda:0", uniform=False)
    db.sides[8] = 3                                   # out of range
    db.sides[9] = 129
    db.sigma[10] = -1.0
    db.pixels[int(b.offsets[11])] = float("nan")
    small, large = db, _repeat(shape, db, 65537)
    got = []
    for batch in (small, large):
        rec, it, st = shape.centroid(batch)
        m, itm, stm = shape.moments(batch, rec)
        torch.cuda.synchronize()
        got.append([t[:db.n].cpu().numpy() for t in (rec, it, st, m, itm, stm)])
    assert (got[0][2][8:11] == shape.ST_BAD_INPUT).all()
    assert got[0][2][11] == shape.ST_NONFINITE_INPUT
    for a, c in zip(*got):
        np.testing.assert_array_equal(a, c)


def _one_side(shape, side, storage, model):
    """24 stamps of one side cut around the galaxies (or stars) of larger ones,
    tiled to a batch beyond the split fit's limit."""
    import torch
    src = synth.make("stars32" if model else "sersic64", count=24)
    w = int(src.sides[0])
    rng = np.random.default_rng(side)
    img = src.pixels.reshape(24, w, w).astype(np.float32)
    pix = 10.0 + rng.normal(0, 1.0, (24, side, side)).astype(np.float32) * src.sigma[:24, None, None]
    a, c = max(0, (w - side) // 2), max(0, (side - w) // 2)
    m = min(w, side)
    pix[:, c:c + m, c:c + m] = img[:, a:a + m, a:a + m]
    scale = None
    if storage == "f16":
        scale = np.exp2(np.ceil(np.log2(np.abs(pix).reshape(24, -1).max(1) / 32768.0)))
        scale = scale.astype(np.float32)
        pix = (pix / scale[:, None, None]).astype(np.float16)
    out = []
    for k in (1, SPLIT_LIMIT // 24 + 1):
        t = lambda x: torch.from_numpy(np.tile(x, (k,) + (1,) * (x.ndim - 1))).cuda()   # noqa: E731
        out.append(shape.DeviceBatch(
            pixels=t(pix).reshape(-1), sigma=t(src.sigma[:24].astype(np.float32)), side0=side,
            scale=None if scale is None else t(scale),
            model=t(np.full(24, model, np.uint8)) if model else None))
    return out


SPLIT_LIMIT = 8192   # (the library's limits are not above this)


def _same_fits(shape, small, large, opts):
    import torch
    got = []
    for batch in (small, large):
        rec0, _, _ = shape.centroid(batch)
        rec, _, _ = shape.moments(batch, rec0)
        f = shape.fit_sersic(batch, rec=rec, opts=opts, want_perr=True)
        torch.cuda.synchronize()
        got.append({k: v[:small.n].cpu().numpy() for k, v in f.items()})
    for k in got[0]:
        np.testing.assert_array_equal(got[0][k], got[1][k], err_msg=k)
    return got[0]


# Every layout of a sweep at the ends of its range: sides 8 to 64 that divide
# 64 (columns; 1, 4, 16 and 64 steps), other sides up to 64 (the walk; one
# step, a ragged last one, several chunks), sides above (segments).
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("side,model", [(8, 0), (16, 0), (32, 0), (64, 0), (4, 0), (7, 0), (33, 0),
                                        (48, 0), (63, 0), (65, 0), (96, 0), (128, 0), (32, 1),
                                        (47, 1), (81, 1)])
def test_split_fit_equals_one_wave_fit(shape, side, model, storage):
    """Four waves per stamp against one wave per stamp (a larger batch)."""
    small, large = _one_side(shape, side, storage, model)
    for kw in (dict(), dict(free_mask=shape.MASK_SIZE),
               dict(free_mask=shape.MASK_SIZE, linear_init=0), dict(max_iter_lm=1)):
        if model and "linear_init" in kw:
            continue
        r = _same_fits(shape, small, large, shape.default_opts(**kw))
        if side >= 32 and not kw:
            assert ((r["status"] & shape.ST_CONVERGED) != 0).sum() >= 12


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_split_fit_of_mixed_sides_and_models(shape, storage):
    b = synth.make("uneven", count=512, storage=storage)
    db = shape.DeviceBatch.from_host(b, "cuda:0", uniform=False)
    db.sides[8] = 3
    db.sigma[10] = -1.0
    db.pixels[int(b.offsets[11])] = float("nan")
    _same_fits(shape, db, _repeat(shape, db, SPLIT_LIMIT + 1), shape.default_opts())


# The one-wave fit drops the model's floor from its sweeps where no pixel can
# reach it; the four-wave fit never does.  Centres on a pixel, near one, half way
# and outside, ellipticities up to the bound, by starting point.
@pytest.mark.parametrize("side", [16, 33, 48, 64, 72])
def test_sweep_without_floor_equals_sweep_with_it(shape, side):
    import torch
    small, large = _one_side(shape, side, "f32", 0)
    rng = np.random.default_rng(side)
    p = np.empty((24, 8), np.float32)
    p[:, 0] = side // 2 + np.tile([0.0, 1e-4, 1e-3, 0.01, 0.5, -side], 4)
    p[:, 1] = side // 2 + np.repeat([0.0, 1e-4, 0.3, 0.5], 6)
    e = np.repeat([0.0, 0.5, 0.99, 0.997], 6)
    th = rng.uniform(0, 2 * np.pi, 24)
    p[:, 2], p[:, 3] = e * np.cos(th), e * np.sin(th)
    p[:, 4:] = [0.15 * side, 2.0, 50.0, 10.0]
    got = []
    for batch in (small, large):
        t = torch.from_numpy(np.tile(p, (batch.n // 24, 1))).cuda()
        f = shape.fit_sersic(batch, p_init=t, opts=shape.default_opts(max_iter_lm=2), want_perr=True)
        got.append({k: v[:24].cpu().numpy() for k, v in f.items()})
    for k in got[0]:
        np.testing.assert_array_equal(got[0][k], got[1][k], err_msg=k)


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("side", [4, 5, 8, 16, 17, 22, 31, 32, 33, 48, 63, 64, 65, 96, 97, 128])
def test_centroid_start_is_the_first_maximum(shape, side, storage):
    """The start before any step: the lowest index among equal maxima, and r50 of
    the growth curve about it (rings ceil(distance), ring 0 within ring 1)."""
    import torch
    rng = np.random.default_rng(side)
    n = 12
    img = rng.integers(0, 4, (n, side, side)).astype(np.float32)   # many equal maxima
    img[0] = 1.0                                                   # nothing above the border
    img[1:5] *= -1.0
    for k, (i, j) in enumerate([(0, 0), (0, side - 1), (side - 1, 0), (side - 1, side - 1)]):
        img[5 + k, i, j] = 9.0
    img[9, side // 2:] = 9.0                                       # whole rows
    img[10, -1, -1], img[11, 0, 0] = np.nan, -np.inf
    pix = torch.from_numpy(img.astype(np.float16) if storage == "f16" else img).cuda().reshape(-1)
    db = shape.DeviceBatch(pixels=pix, sigma=torch.ones(n, device="cuda"), side0=side,
                           scale=torch.ones(n, device="cuda") if storage == "f16" else None)
    rec, it, st = (t.cpu().numpy() for t in shape.centroid(db, shape.default_opts(max_iter_centroid=0)))
    assert (st[10:] == shape.ST_NONFINITE_INPUT).all() and np.isnan(rec[10:]).all()
    assert (it == 0).all()
    ii, jj = np.mgrid[:side, :side]
    for s in range(10):
        a = img[s].astype(np.float64)
        i0, j0 = divmod(int(np.argmax(a)), side)
        assert (rec[s, 0], rec[s, 1]) == (j0, i0), s   # x0, y0; 5 is r50, 7 the flux
        edge = np.concatenate([a[0], a[-1], a[1:-1, 0], a[1:-1, -1]])
        f = a - edge.sum() / (4.0 * side - 4.0)
        ring = np.ceil(np.sqrt((ii - i0) ** 2 + (jj - j0) ** 2)).astype(int)
        c = np.cumsum(np.bincount(ring.ravel(), weights=f.ravel()))
        if abs(c[-1]) < 1e-9 * np.abs(f).sum() + 1e-9:
            continue   # the total's sign is its rounding's
        if c[-1] < 0:
            assert st[s] & shape.ST_NONPOSITIVE_FLUX
            continue
        r = int(np.argmax((2 * c >= c[-1]) & (np.arange(len(c)) >= 1)))
        before = 0.0 if r == 1 else c[r - 1]
        want = (r - 1) + (0.5 * c[-1] - before) / (c[r] - before)
        # FP64 sums of up to 2^14 terms against an exact total, then FP32
        np.testing.assert_allclose(rec[s, 5], want, rtol=1e-6, atol=1e-6)
        np.testing.assert_allclose(rec[s, 7], c[-1], rtol=1e-6)


def _time(f, repeat=5):
    """Shortest of `repeat` passes, in ms."""
    import torch
    f()
    best = float("inf")
    for _ in range(repeat):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 4)
    return best


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_fit_of_some_split_stamps(shape, storage):
    """1,000 stamps of mixed sides, of which the largest take four waves each,
    against one wave each (a larger batch)."""
    b = synth.make("uneven", count=1000, storage=storage)
    db = shape.DeviceBatch.from_host(b, "cuda:0", uniform=False)
    assert b.sides.max() > 1.5 * np.sqrt(np.mean(b.sides.astype(float) ** 2)) + 8
    db.sides[8] = 3
    db.sigma[10] = -1.0
    db.pixels[int(b.offsets[11])] = float("nan")
    large = _repeat(shape, db, SPLIT_LIMIT + 1)
    for kw in (dict(), dict(free_mask=shape.MASK_SIZE), dict(max_iter_lm=1)):
        _same_fits(shape, db, large, shape.default_opts(**kw))
    db.model = large.model = None
    _same_fits(shape, db, large, shape.default_opts(free_mask=shape.MASK_SIZE, linear_init=0))


def test_stamps_of_equal_sides_cost_the_same_with_a_side_array(shape):
    """Of 4,096 stamps of 24 x 24 none sets the pace: given with offsets and sides
    (as cut-outs are) they take little more than a batch of one side (1.23 times;
    four waves for each stamp took 2.16 times)."""
    import torch
    b = synth.make("sersic64", count=64)
    w, side, n = int(b.sides[0]), 24, 4096
    c = (w - side) // 2
    img = b.pixels.reshape(64, w, w)[:, c:c + side, c:c + side].astype(np.float32)
    pix = torch.from_numpy(np.ascontiguousarray(img)).cuda().repeat(n // 64, 1, 1).reshape(-1)
    sigma = torch.from_numpy(b.sigma[:64].astype(np.float32)).cuda().repeat(n // 64)
    one = shape.DeviceBatch(pixels=pix, sigma=sigma, side0=side)
    sided = shape.DeviceBatch(pixels=pix, sigma=sigma,
                              offsets=torch.arange(n, device="cuda") * side * side,
                              sides=torch.full((n,), side, dtype=torch.int32, device="cuda"))
    rec, _, _ = shape.moments(one, shape.centroid(one)[0])
    t1 = _time(lambda: shape.fit_sersic(one, rec=rec))
    t2 = _time(lambda: shape.fit_sersic(sided, rec=rec))
    assert t2 < 1.6 * t1, (t1, t2)


@pytest.mark.parametrize("n", [16384, 16385, 49152, 49153])
def test_mixed_sides_at_the_limits_of_one_launch(shape, n):
    """The last batch that centroid (49,152) and moments (16,384) take in one
    launch, and the first of a launch per form, against a small one."""
    import torch
    b = synth.make("uneven", count=256)
    db = shape.DeviceBatch.from_host(b, "cuda:0", uniform=False)
    db.sides[8], db.sigma[10] = 3, -1.0
    got = []
    for batch in (db, _repeat(shape, db, n)):
        rec, it, st = shape.centroid(batch)
        out = (rec, it, st) + tuple(shape.moments(batch, rec))
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in out])
    idx = np.arange(n) % db.n
    for a, c in zip(*got):
        np.testing.assert_array_equal(c, a[idx])
