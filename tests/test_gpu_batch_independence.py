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
