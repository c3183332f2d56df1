"""GPU: the first launch of a scan, which clears the accumulator and the
counters, makes the primaries and, for one scan without a mask whose tables
fit its arguments (58 materials), brings the tables."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2310_03505_amd as lib
    lib.load_library()
    return lib


@pytest.mark.parametrize("n_mats", [2, 58, 59, 200])
@pytest.mark.parametrize("n_az, rays, bins", [
    (1, 1, 1),          # fewer items than counters
    (3, 5, 60000),     # far more cells than primaries
    (1, 3001, 7),       # more primaries than cells
    (400, 64, 512),
])
def test_first_launch_forms_agree(R, n_mats, n_az, rays, bins):
    """The same scan through every form of the first launch, each on scratch
    memory that a larger scan left full: alone (tables in the arguments, or
    put first above 58 materials), with a mask of ones (separate clear), as
    the second of a batch, and replayed in a graph.  Accumulators, images and
    records are equal bit for bit, and the masked form was there before."""
    import torch
    s = W.tiny_room(n_azimuth=n_az, rays_per_beam=rays, beam_width_deg=20.0)
    s.params.update(n_bins=bins, bin_size_m=22.5 / bins)
    big = W.tiny_room(n_azimuth=401, rays_per_beam=65, beam_width_deg=20.0)
    big.params.update(n_bins=1000, bin_size_m=0.02)
    used = len(s.materials)
    mats = [s.materials[i % used] for i in range(max(n_mats, used))]
    ctx = R.Context(0)
    sc = R.Scene(ctx, s.vertices, s.indices, s.tri_material)
    try:
        dirty = lambda: R.rr_radar_scan_batch(ctx.handle, sc.handle, [(big.pose, big.params)] * 2, mats)
        dirty()
        ones = torch.ones(n_az * rays, dtype=torch.uint8, device="cuda")
        want = R.rr_radar_scan_records(ctx.handle, sc.handle, s.pose, s.params, mats, primary_mask=ones)
        for _ in range(2):
            dirty()
            got = R.rr_radar_scan_records(ctx.handle, sc.handle, s.pose, s.params, mats)
            for k in ("image", "records", "accum"):
                assert torch.equal(got[k], want[k]), k
            assert got["stats"]["rays_per_depth"] == want["stats"]["rays_per_depth"]
        dirty()
        images, _ = R.rr_radar_scan_batch(ctx.handle, sc.handle, [(big.pose, big.params), (s.pose, s.params)], mats)
        assert torch.equal(images[1], want["image"])
        g, out = R.rr_graph_create(ctx.handle, sc.handle, [(s.pose, s.params)], mats)
        try:
            for _ in range(3):
                dirty()
                out[0].zero_()
                R.rr_graph_launch(g)
                torch.cuda.synchronize()
                assert torch.equal(out[0], want["image"])
        finally:
            R.rr_graph_destroy(g)
    finally:
        sc.release()
        ctx.close()


@pytest.mark.parametrize("n_az", [256, 1536])
@pytest.mark.parametrize("more", [0, 1])
def test_shade_block_sizes_agree(R, n_az, more):
    """Levels at and just above the sizes where the interaction's blocks grow
    (256 and 1,536 rays per compute unit): the scan alone and as one of a
    batch that runs the largest blocks gives the same image bit for bit, with
    the same rays."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    s = W.tiny_room(n_azimuth=n_az, rays_per_beam=n_cu + more, beam_width_deg=20.0, max_bounces=3)
    ctx = R.Context(0)
    sc = R.Scene(ctx, s.vertices, s.indices, s.tri_material)
    try:
        alone, st = R.rr_radar_scan(ctx.handle, sc.handle, s.pose, s.params, s.materials, stats=True)
        n = -(-4 * 1536 // n_az)
        images, bst = R.rr_radar_scan_batch(ctx.handle, sc.handle, [(s.pose, s.params)] * n, s.materials, stats=True)
        torch.cuda.synchronize()
        assert st["overflow"] == 0 and bst["overflow"] == 0
        assert all(torch.equal(i, alone) for i in images)
        assert bst["rays_per_depth"] == [n * r for r in st["rays_per_depth"]]
        assert float(alone.max()) > 0
    finally:
        sc.release()
        ctx.close()
