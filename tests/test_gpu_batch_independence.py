"""GPU: what is computed for a frame or a stamp does not depend on what else is
in the call (how many there are, how large the buffer is), bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shape():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1203_0571_amd as shape
    return shape


def _cancelling_frames(n, H, W, f16):
    """Frames of pixels over 40 binary orders whose sum cancels, so that every
    rounding of the sums shows in F and r50."""
    rng = np.random.default_rng(H * W)
    scale = None
    inner = (H - 2) * (W - 2) // 2 * 2
    pix = np.zeros((n, H, W), np.float32)
    for k in range(n):
        a = np.exp2(rng.uniform(-24, 15, inner // 2) if f16 else rng.uniform(-20, 20, inner // 2))
        v = rng.permutation(np.concatenate([a, -a]).astype(np.float16 if f16 else np.float32))
        box = np.zeros((H - 2) * (W - 2), np.float32)
        box[:inner] = v
        pix[k, 1:-1, 1:-1] = box.reshape(H - 2, W - 2)
    if f16:
        pix, scale = pix.astype(np.float16), np.full(n, 0.3, np.float32)
    return pix, scale


def _detect(shape, pix, scale):
    import torch
    d = shape.frame_detect(shape.DeviceFrames(pixels=pix, scale=scale))
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in d.items()}


@pytest.mark.parametrize("f16", [False, True])
def test_a_frame_alone_and_among_many(shape, f16):
    """3 frames, and the same 70 times over: sums of 517 x 333 pixels."""
    import torch
    pix, scale = _cancelling_frames(3, 517, 333, f16)
    t = torch.from_numpy(pix).cuda()
    s = None if scale is None else torch.from_numpy(scale).cuda()
    few = _detect(shape, t, s)
    many = _detect(shape, t.repeat(70, 1, 1), None if s is None else s.repeat(70))
    assert (few["info"][:, 2] != 0.0).any()
    for k, v in few.items():
        np.testing.assert_array_equal(many[k].reshape((70,) + v.shape),
                                      np.broadcast_to(v, (70,) + v.shape), err_msg=k)


def _perfect_stamps(shape, side, f16, n=12):
    """Stamps that hold their model to the last bit of the pixels, so that r is
    rounding alone and the sums show every change of it."""
    import oracle
    rng = np.random.default_rng(side)
    c = 0.5 * (side - 1)
    p = np.empty((n, 8))
    p[:, 0:2] = c + rng.uniform(-0.9, 0.9, (n, 2))
    p[:, 2:4] = rng.uniform(-0.3, 0.3, (n, 2))
    p[:, 4] = rng.uniform(0.08, 0.3, n) * side
    p[:, 5] = rng.uniform(0.5, 5.0, n)
    p[:, 6] = rng.uniform(1.0, 100.0, n)
    p[:, 7] = rng.uniform(-5.0, 5.0, n)
    p = p.astype(np.float32)
    img = np.stack([oracle.model(side, q) for q in p.astype(np.float64)]).reshape(n, -1)
    return p, (img * 2.0).astype(np.float16) if f16 else img.astype(np.float32)


@pytest.mark.parametrize("f16", [False, True])
@pytest.mark.parametrize("side", [12, 16, 32, 47, 48, 64])
def test_chi2_of_a_stamp_alone_and_among_many(shape, side, f16):
    """12 stamps; the same in a batch of over 3e7 pixels; with a side array, alone
    and in a buffer of 128 x 128 pixels a stamp, beside larger stamps."""
    import torch
    p, pix = _perfect_stamps(shape, side, f16)
    n, area = len(p), side * side
    t, pt = torch.from_numpy(pix).cuda(), torch.from_numpy(p).cuda()

    def batch(pixels, k, **kw):
        return shape.DeviceBatch(pixels=pixels, sigma=torch.full((k,), 1e-6, device="cuda"),
                                 scale=torch.full((k,), 0.5, device="cuda") if f16 else None, **kw)

    def outputs(db, params, pick):
        out = dict(value=shape.chi2_fwd(db, params))
        for want in (False, True):
            for key, v in shape.chi2_bwd(db, params, want_normal=want).items():
                if v is not None:
                    out["%s %d" % (key, want)] = v
        return {key: v[pick].cpu().numpy() for key, v in out.items()}

    alone = outputs(batch(t.reshape(-1), n, side0=side), pt, slice(0, n))
    k = 30_000_000 // (n * area) + 1
    many = outputs(batch(t.repeat(k, 1).reshape(-1), n * k, side0=side), pt.repeat(k, 1),
                   slice(n * (k - 1), n * k))
    i = torch.arange(n, device="cuda")
    sided = outputs(batch(t.reshape(-1), n, offsets=i * area, sides=(i * 0 + side).int()), pt,
                    slice(0, n))
    # the stamps first, then as many again of 128 x 128
    big = torch.zeros(2 * n * 128 * 128, dtype=t.dtype, device="cuda")
    big[:n * area] = t.reshape(-1)
    mixed = outputs(batch(big, 2 * n, offsets=torch.cat([i * area, n * area + i * 128 * 128]),
                          sides=torch.cat([i * 0 + side, i * 0 + 128]).int()),
                    pt.repeat(2, 1), slice(0, n))
    for key, v in alone.items():
        np.testing.assert_array_equal(many[key], v, err_msg=key)
        np.testing.assert_array_equal(mixed[key], sided[key], err_msg=key)
