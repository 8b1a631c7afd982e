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
