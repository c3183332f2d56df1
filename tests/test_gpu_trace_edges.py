"""GPU: the closest-hit launch at the sizes where its work split changes."""
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


def _records(R, ctx, sc, s, p):
    import torch
    o = R.rr_radar_scan_records(ctx.handle, sc.handle, s.pose, p, s.materials)
    torch.cuda.synchronize()
    return o


@pytest.mark.parametrize("rays", [1, 63, 64, 65, 129, 16383, 16384, 16385, 16449, 33001])
def test_ray_shares_and_claims(R, ctx, rays):
    """Every wave starts with a share of the queue and claims the rest: one
    wave per compute unit gives a grid of 16,384 lanes (256 units), so these
    queues lie below, at and above one ray per lane, with shares of 1 to 64
    rays and dynamic parts of 0, 1, 65 and many rays.  Path records of every
    non-exempt primary equal the oracle's; the default grid, the one-launch
    form and the eight-wide tree give the same records and accumulator bit
    for bit."""
    import torch
    s = W.tiny_room(n_azimuth=1, rays_per_beam=rays, beam_width_deg=40.0)
    before = R.rr_get_tuning(ctx.handle)
    sc = R.Scene(ctx, s.vertices, s.indices, s.tri_material)
    sc8 = R.Scene(ctx, s.vertices, s.indices, s.tri_material, width=8)
    try:
        R.rr_set_tuning(ctx.handle, **dict({k: before[k] for k in R.TUNING_KEYS}, trace_waves_per_cu=1))
        outs = [_records(R, ctx, sc, s, s.params), _records(R, ctx, sc8, s, s.params)]
        R.rr_set_tuning(ctx.handle, **dict({k: before[k] for k in R.TUNING_KEYS}, trace_waves_per_cu=1, fused=1))
        outs.append(_records(R, ctx, sc, s, s.params))
        R.rr_set_tuning(ctx.handle, **{k: before[k] for k in R.TUNING_KEYS})
        outs.append(_records(R, ctx, sc, s, s.params))
    finally:
        R.rr_set_tuning(ctx.handle, **{k: before[k] for k in R.TUNING_KEYS})
        sc.release()
        sc8.release()
    for o in outs[1:]:
        assert torch.equal(o["records"], outs[0]["records"])
        assert torch.equal(o["accum"], outs[0]["accum"])
    ref = oracle.scan_scene(s, records=True, exempt=True)
    ok = ~ref["exempt"]
    assert (outs[0]["records"].cpu().numpy()[ok] == ref["records"][ok]).all()
    assert ok.mean() > 0.98 or rays < 100
    assert np.isfinite(outs[0]["image"].cpu().numpy()).all()


@pytest.mark.parametrize("size, bin_size, index", [
    (1.0, 0.044, 0.5),      # a medium thinner than air: the ray's limit exceeds the sensor's range
    (1.0, 1e30, 2.5),       # limits near the top of float32
    (1.0, 1e-25, 2.5),      # a range far below any distance: no hit at all
    (1.5e6, 6.6e4, 2.5),    # coordinates near the largest accepted
    (2e-3, 8.8e-5, 2.5),    # a scene of centimetres
])
def test_box_tests_at_range_extremes(R, ctx, size, bin_size, index):
    """Box tests work in distances scaled by a power of two per ray; whatever
    the scale, the closest hits are the oracle's brute-force ones (every
    non-exempt primary) and equal the eight-wide traversal's, which does not
    scale."""
    import torch
    s = W.tiny_room(n_azimuth=100, rays_per_beam=24, max_bounces=4)
    s.vertices = (s.vertices * np.float32(size)).astype(np.float32)
    s.params = dict(s.params, bin_size_m=bin_size)
    s.materials = [dict(m, n=index) if m["kind"] == W.KIND_DIELECTRIC else m for m in s.materials]
    outs = []
    for opts in (dict(), dict(width=8), dict(builder=1)):
        sc = R.Scene(ctx, s.vertices, s.indices, s.tri_material, **opts)
        try:
            outs.append(_records(R, ctx, sc, s, s.params))
        finally:
            sc.release()
    for o in outs[1:]:
        assert torch.equal(o["records"], outs[0]["records"])
        assert torch.equal(o["accum"], outs[0]["accum"])
    ref = oracle.scan_scene(s, records=True, exempt=True)
    ok = ~ref["exempt"]
    assert (outs[0]["records"].cpu().numpy()[ok] == ref["records"][ok]).all()
    hits = (ref["records"] >= 0).sum()
    assert (hits == 0) == (bin_size < 1e-20)
