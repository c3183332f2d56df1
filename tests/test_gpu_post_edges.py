"""GPU: the epilogue's logarithm table and load paths at their edges."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2310_03505_amd as lib
    lib.load_library()
    return lib


@pytest.fixture(scope="module")
def ctx(R):
    c = R.Context(0)
    yield c
    c.close()


def _edge_values():
    # the 128 table intervals' borders (exact in float32) and their
    # neighbours, over the float32 exponents; around 1; specials
    hi = (0x3fe60000 + (np.arange(129, dtype=np.uint64) << np.uint64(13))) << np.uint64(32)
    z = hi.view(np.float64).astype(np.float32)
    z = np.concatenate([np.nextafter(z, np.float32(0)), z, np.nextafter(z, np.float32(9))])
    v = [np.ldexp(z, k).astype(np.float32) for k in (-140, -126, -60, -20, -1, 0, 1, 40, 127)]
    one = np.float32(1)
    steps = np.arange(1, 65, dtype=np.float32)
    v += [one + steps * np.float32(2.0 ** -23), one - steps * np.float32(2.0 ** -24)]
    v += [np.array([0.0, -0.0, -1.0, -np.inf, np.inf, np.nan, 1.0, 1e-45, 3.4e38], np.float32)]
    return np.concatenate(v)


@pytest.mark.parametrize("pad", [0, 1, 2, 3])
def test_db_at_table_borders(R, ctx, pad):
    """dB of values at and next to every border of the logarithm table, at the
    ends of float32, around 1 (where the result keeps its relative accuracy)
    and of special values: within one float32 ulp of numpy's float64, 8-bit
    pixels exact except within 1e-9 of a rounding boundary; row lengths of
    every remainder by four (one load per four pixels, or four)."""
    import torch
    with np.errstate(over="ignore", invalid="ignore", divide="ignore"):
        x = _edge_values()
        x = np.concatenate([x, np.full((-len(x)) % 4 + pad, 0.5, np.float32)])
        db, u8 = R.rr_postprocess(ctx.handle, torch.from_numpy(x[None]).cuda(), dict())
        db, u8 = db.cpu().numpy()[0], u8.cpu().numpy()[0]
        pos = x > 0
        want = np.where(pos, 10.0 * np.log10(np.where(pos, x, 1.0).astype(np.float64)), -np.inf)
    fin = np.isfinite(want)
    assert np.array_equal(db[~fin], want[~fin].astype(np.float32))
    w32 = want[fin].astype(np.float32)
    assert (np.abs(db[fin].astype(np.float64) - w32) <= np.spacing(np.abs(w32)).astype(np.float64)).all()
    pre = np.where(fin, 255.0 * (np.where(fin, want, 0.0) + 100.0) / 100.0, np.where(want > 0, 1e9, -1e9))
    ok = np.abs(pre + 0.5 - np.round(pre + 0.5)) >= 1e-9
    assert (u8[ok] == np.clip(np.floor(pre + 0.5), 0, 255)[ok]).all()


@pytest.mark.parametrize("shape", [(1, 3, 1024), (2, 5, 1028), (1, 2, 3776), (1, 4, 1025)])
def test_unaligned_images(R, ctx, shape):
    """Images that start off a 16-byte boundary take four loads per lane
    instead of one: same pixels, bit for bit, and the oracle's."""
    import torch
    post = dict(blur_sigma_bins=2.0, uniform_amp=1e-7, perlin_amp=1e-6, perlin_cell_az=16.0, perlin_cell_bins=64.0,
                seed=5)
    imgs = W.polar_images(3, *shape)
    flat = torch.from_numpy(np.concatenate([np.zeros(1, np.float32), imgs.reshape(-1)])).cuda()
    a = R.rr_postprocess(ctx.handle, torch.from_numpy(imgs).cuda(), post)
    b = R.rr_postprocess(ctx.handle, flat[1:].view(shape), post)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    _, u8, pre = oracle.postprocess(imgs[0], post)
    off = np.abs(pre - (np.floor(pre) + 0.5)) < 1e-9
    assert ((a[1][0].cpu().numpy() == u8) | off).all()
