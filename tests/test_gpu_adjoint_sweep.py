"""GPU: the FP64 sweep behind chi2_fwd / chi2_bwd over its pixel layouts (how a
side is cut into runs of rows) and its two series (tabulated powers; the full
series for stamps the tables do not cover), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_adjoint import _check_grad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shape():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_0571_amd as shape
    return shape


def _stamps(side, storage, n=16):
    """Stamps of noise and parameters; from stamp 10 on ones the tables miss."""
    rng = np.random.default_rng(side)
    c = 0.5 * (side - 1)
    p = np.empty((n, 8))
    p[:, 0:2] = c + rng.uniform(-0.9, 0.9, (n, 2))
    r, th = rng.uniform(0, 0.7, n), rng.uniform(0, 2 * np.pi, n)
    p[:, 2], p[:, 3] = r * np.cos(th), r * np.sin(th)
    p[:, 4] = rng.uniform(0.08, 0.3, n) * side
    p[:, 5] = rng.uniform(0.4, 6.0, n)
    p[:, 6] = rng.uniform(1.0, 100.0, n)
    p[:, 7] = rng.uniform(-5.0, 5.0, n)
    p[0, 0] = -2.25                 # the centre outside the stamp
    p[10, 0:2] = np.floor(c)        # on a pixel: the model's floor
    p[11, 2:4] = 0.9995, 0.0        # |e| beyond the tables' range
    p[12, 4] = 2e5                  # Re beyond it
    p[13, 0:2] = np.floor(c) + [1e-4, 0.0]   # R^2 below it
    p[14, 2] = np.nan
    p = p.astype(np.float32).astype(np.float64)
    pix = rng.normal(3.0, 2.0, (n, side, side)).astype(np.float32)
    if storage == "f16":
        pix = pix.astype(np.float16)
    return p, pix, rng.uniform(1.0, 3.0, n).astype(np.float32)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("side", [4, 5, 8, 16, 31, 33, 48, 63, 64, 65, 100, 128])
def test_sersic_sweep_vs_oracle(shape, side, storage, large):
    """Outputs are FP64 sums (series good to 5e-14) rounded to FP32 (6e-8): 1e-6
    of each, and of entries down to 1e-3 of the largest where terms cancel.
    large: a batch of 3e7 pixels, which takes the tables at every side."""
    import torch
    p, pix, sigma = _stamps(side, storage)
    n = len(p)
    k = 30_000_000 // (n * side * side) + 1 if large else 1
    db = shape.DeviceBatch(pixels=torch.from_numpy(pix).cuda().reshape(-1).repeat(k),
                           sigma=torch.from_numpy(sigma).cuda().repeat(k), side0=side,
                           scale=torch.full((n * k,), 0.5, device="cuda") if storage == "f16" else None)
    pt = torch.from_numpy(p.astype(np.float32)).cuda().repeat(k, 1)

    def first(t):   # every copy of the stamps gives the same bits
        a = t.reshape((k, n) + t.shape[1:])
        assert bool(((a == a[:1]) | ((a != a) & (a[:1] != a[:1]))).all())
        return a[0].cpu().numpy()
    value = first(shape.chi2_fwd(db, pt))
    plain = {q: first(v) for q, v in shape.chi2_bwd(db, pt).items() if v is not None}
    full = {q: first(v) for q, v in shape.chi2_bwd(db, pt, want_normal=True).items()}
    img = pix.astype(np.float64) * (0.5 if storage == "f16" else 1.0)
    for out in (value, plain["chi2"], plain["grad"], full["grad"], full["jtj"]):
        assert np.isnan(out[14]).all()
    np.testing.assert_array_equal(plain["chi2"], value)
    np.testing.assert_array_equal(full["chi2"], value)
    for s in range(n):
        if s == 14:
            continue
        c2, g, jtj = oracle.chi2(img[s], float(sigma[s]), p[s], want_grad=True)
        assert abs(value[s] / c2 - 1) < 1e-6, s
        for got in (plain, full):
            err = _check_grad(got["grad"][s:s + 1].astype(np.float64), g[None], p[s:s + 1], sigma[s:s + 1])
            assert err < 1e-6, (s, err)
        # entry (k, l) in units of its columns' norms, the diagonal
        d = np.sqrt([jtj[k * 8 - k * (k - 1) // 2] for k in range(8)])
        unit = np.array([d[k] * d[m] for k in range(8) for m in range(k, 8)])
        assert (np.abs(full["jtj"][s] - jtj) <= 1e-6 * np.maximum(np.abs(jtj), 1e-3 * unit)).all(), s


def test_chunks_of_stamps_do_not_change_the_results(shape):
    """A workgroup takes several stamps of a large batch and one of a small one,
    skipping the other model's."""
    import torch
    p, pix, sigma = _stamps(48, "f32")
    model = np.zeros(len(p), np.uint8)
    model[3::4] = 1
    p[3::4, 5] = 3.0
    out = []
    for k in (1, 1025):     # 16 and 16,400 stamps
        t = lambda x: torch.from_numpy(np.tile(x, (k,) + (1,) * (x.ndim - 1))).cuda()   # noqa: E731
        db = shape.DeviceBatch(pixels=t(pix).reshape(-1), sigma=t(sigma), side0=48, model=t(model))
        out.append(shape.chi2_bwd(db, t(p.astype(np.float32)), want_normal=True))
    for key in ("chi2", "grad", "jtj"):
        small, large = (o[key].cpu().numpy() for o in out)
        np.testing.assert_array_equal(large.reshape((1025,) + small.shape),
                                      np.broadcast_to(small, (1025,) + small.shape))


# Stamps at the ends of what the tables cover: ellipticity, index and size, the
# cut at b t = 740 (small sizes and indices), a centre far off and one just above
# the smallest R^2.  (x0, y0 from the middle pixel; e1, e2; Re; n.)
TABLE_ENDS = [(0.3, 0.4, 0.95, 0.0, 9.0, 2.0), (0.3, 0.4, 0.0, -0.95, 9.0, 0.6),
              (0.45, 0.35, 0.998, 0.0, 9.0, 1.0), (0.45, 0.35, -0.7, 0.711, 9.0, 4.0),
              (0.3, 0.4, 0.2, 0.1, 9.0, 0.15), (0.3, 0.4, 0.2, 0.1, 9.0, 18.0),
              (0.3, 0.4, 0.2, 0.1, 0.002, 4.0), (0.3, 0.4, 0.2, 0.1, 0.05, 0.5),
              (0.3, 0.4, 0.2, 0.1, 0.3, 0.2), (0.3, 0.4, 0.2, 0.1, 9e4, 1.0),
              (0.3, 0.4, 0.2, 0.1, 9e4, 0.3), (-4000.3, 700.4, 0.2, 0.1, 900.0, 1.5),
              (4e-4, 0.0, 0.0, 0.0, 9.0, 1.0), (4e-4, 0.0, 0.0, 0.0, 9.0, 6.0)]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("side", [48, 64, 100])
def test_sersic_tables_at_the_ends_of_their_range(shape, side, storage):
    """1e-6 as above (at |e| = 0.998 the quadratics of R^2 would cancel to 1e-16 (2 /
    0.002)^2 = 1e-10), beside FP32's smallest normal number, 1.2e-38."""
    import torch
    n = len(TABLE_ENDS)
    rng = np.random.default_rng(side)
    p = np.empty((n, 8))
    p[:, :6] = TABLE_ENDS
    p[:, 0:2] += side // 2
    p[:, 6] = rng.uniform(1.0, 100.0, n)
    p[:, 7] = rng.uniform(-5.0, 5.0, n)
    p = p.astype(np.float32).astype(np.float64)
    pix = rng.normal(3.0, 2.0, (n, side, side)).astype(np.float16 if storage == "f16" else np.float32)
    sigma = rng.uniform(1.0, 3.0, n).astype(np.float32)
    db = shape.DeviceBatch(pixels=torch.from_numpy(pix).cuda().reshape(-1),
                           sigma=torch.from_numpy(sigma).cuda(), side0=side,
                           scale=torch.full((n,), 0.5, device="cuda") if storage == "f16" else None)
    pt = torch.from_numpy(p.astype(np.float32)).cuda()
    value = shape.chi2_fwd(db, pt).cpu().numpy()
    got = {k: v.cpu().numpy() for k, v in shape.chi2_bwd(db, pt, want_normal=True).items()}
    img = pix.astype(np.float64) * (0.5 if storage == "f16" else 1.0)
    for s in range(n):
        c2, g, jtj = oracle.chi2(img[s], float(sigma[s]), p[s], want_grad=True)
        assert abs(value[s] / c2 - 1) < 1e-6, s
        err = _check_grad(got["grad"][s:s + 1].astype(np.float64), g[None], p[s:s + 1], sigma[s:s + 1])
        assert err < 1e-6, (s, err)
        d = np.sqrt([jtj[k * 8 - k * (k - 1) // 2] for k in range(8)])
        unit = np.array([d[k] * d[m] for k in range(8) for m in range(k, 8)])
        tol = 1e-6 * np.maximum(np.abs(jtj), 1e-3 * unit) + 1.2e-38
        assert (np.abs(got["jtj"][s] - jtj) <= tol).all(), s


def test_bad_stamps_beside_good_ones(shape):
    """Several stamps to a workgroup (over 16,384 of them): those that cannot be
    evaluated give NaN, and their neighbours what they give in a small batch."""
    import torch
    p, pix, sigma = _stamps(48, "f32")
    k = 1025
    t = lambda x: torch.from_numpy(np.tile(x, (k,) + (1,) * (x.ndim - 1))).cuda()   # noqa: E731
    bad = np.zeros(16 * k, bool)
    bad[[0, 7, 8, 4097, 4098, 16 * k - 1]] = True
    good_sigma, model = t(sigma), np.zeros(16 * k, np.uint8)
    bad_sigma = torch.where(torch.from_numpy(bad).cuda(), -good_sigma, good_sigma)
    model[5000] = 7                                     # no such model
    bad[5000] = True
    small = shape.DeviceBatch(pixels=torch.from_numpy(pix).cuda().reshape(-1),
                              sigma=torch.from_numpy(sigma).cuda(), side0=48)
    large = shape.DeviceBatch(pixels=t(pix).reshape(-1), sigma=bad_sigma, side0=48,
                              model=torch.from_numpy(model).cuda())
    par = torch.from_numpy(p.astype(np.float32)).cuda()
    a = shape.chi2_bwd(small, par, want_normal=True)
    b = shape.chi2_bwd(large, par.repeat(k, 1), want_normal=True)
    for key in ("chi2", "grad", "jtj", "jtr"):
        x, y = a[key].cpu().numpy(), b[key].cpu().numpy()
        assert np.isnan(y[bad]).all()
        np.testing.assert_array_equal(y[~bad], x[np.arange(16 * k) % 16][~bad])
