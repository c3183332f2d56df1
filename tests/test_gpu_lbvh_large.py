"""GPU tree build, refit and rebuild beyond one pass of their strided launches.

Launches that give a lane several items take 512 blocks of 1,024 lanes
(524,288 triangles), the node emission 2,048 blocks of 256 (524,288 nodes);
the boxes over the sorted positions are filled nine levels a launch, by three
launches above 262,144 hittable triangles.
"""
import numpy as np
import pytest

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


@pytest.mark.parametrize("n, leaf, degenerate", [
    (262144, 2, False),   # the most that two box launches fill
    (262145, 2, False),   # one more
    (524289, 2, False),   # one triangle in the second pass of the strided launches
    (1500001, 1, True),   # more nodes than lanes of the node emission
])
def test_build_refit_rebuild_large(R, ctx, n, leaf, degenerate):
    """After the build, after a refit, after a rebuild in the arrays of the
    first build and after a refit of that, scans give the records and the
    accumulator of a host-built (and refitted) tree bit for bit, and the tree
    passes the host check where no triangle changed its kind."""
    import torch
    rng = np.random.default_rng(n)
    c = rng.uniform(-6.0, 6.0, (n, 1, 3))
    V = (c + rng.uniform(-0.1, 0.1, (n, 3, 3))).astype(np.float32)
    if degenerate:
        V[3::17, 2] = V[3::17, 1]
    V = V.reshape(-1, 3)
    F = np.arange(3 * n, dtype=np.uint32).reshape(n, 3)
    M = (np.arange(n) % 3).astype(np.uint16)
    mats = W.tiny_room().materials
    p = W.sensor_params(32, 24, 3, 512, beam_width_deg=20.0)
    pose = W.yaw_pose((0.1, -0.2, 0.3), 0.4)
    moves = []
    for k in (1, 2):
        by = np.float32(0.3) * np.sin(V[:, [1, 2, 0]] + np.float32(k))
        moves.append(torch.from_numpy(np.ascontiguousarray(V + by, dtype=np.float32)).cuda())
    hittable = n - (len(range(3, n, 17)) if degenerate else 0)
    host = R.Scene(ctx, V, F, M, spatial_pct=-1)
    sc = R.Scene(ctx, V, F, M, builder=1, max_leaf_size=leaf)
    try:
        def scan(s):
            o = R.rr_radar_scan_records(ctx.handle, s.handle, pose, p, mats)
            torch.cuda.synchronize()
            return o["records"], o["accum"]

        def same(a, b):
            assert (a[0][:, 0] >= 0).float().mean() > 0.5  # enough to compare
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        first = sc.info()
        assert first["n_hittable"] == hittable
        assert (first["n_nodes"] > 524288) == (leaf == 1)
        want = scan(host)
        print("case: build", n, flush=True)
        same(scan(sc), want)
        assert sc.selfcheck(20, n) == 0
        print("case: refit", n, flush=True)
        host.refit(moves[0])
        sc.refit(moves[0])
        same(scan(sc), scan(host))
        if not degenerate:
            assert sc.selfcheck(20, n) == 0
        print("case: rebuild", n, flush=True)
        R.rr_bvh_build(ctx.handle, sc.handle, builder=1, max_leaf_size=leaf)
        same(scan(sc), want)
        again = sc.info()
        assert {k: v for k, v in again.items() if k != "build_ms"} == {k: v for k, v in first.items() if k != "build_ms"}
        print("case: refit of the rebuilt tree", n, flush=True)
        host.refit(moves[1])
        sc.refit(moves[1])
        same(scan(sc), scan(host))
    finally:
        sc.release()
        host.release()
