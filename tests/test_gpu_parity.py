"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle on the same
seeded inputs.  Block key sets (with levels) must be bit-identical, weights exactly equal and
TSDF values within 1e-5 m (FP32 storage against the FP64 oracle)."""
import numpy as np
import pytest
import torch

from parity_util import announce, compare_maps, excused_keys, gpu_sorted
from workloads import configs, room_sequence, sphere_plane_frame, street_sequence

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mrh():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2511_21459_amd as mrh

    return mrh


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_sphere_plane_frame(mrh, orc):
    announce("sphere_plane single frame 320x240")
    depth, cam, T = sphere_plane_frame(seed=0)
    g = mrh.Map(**configs.SPHERE_PLANE)
    g.integrate_depth(_dev(depth), cam.K, T)
    last, _ = g.sync()
    o = orc.OracleMap(**configs.oracle_kwargs(configs.SPHERE_PLANE))
    st = o.integrate_depth(depth, cam.K, T)
    assert last["valid_points"] == st["valid_points"] == 76800
    assert last["new_blocks"] == st["new_blocks"] == o.num_blocks
    assert last["observations"] == st["observations"]
    assert last["distinct_voxels"] == st["distinct_voxels"]
    assert last["candidate_keys"] == st["candidate_keys"]
    rep = compare_maps(gpu_sorted(g), o.extract(), tau=0.06)
    print(rep)


@pytest.mark.parametrize("form", ["range", "zdiff"])
def test_room_sequence_multires(mrh, orc, form):
    """Multi-resolution orbit at reduced size: 320x240, 12 frames spread over the orbit."""
    announce(f"room 320x240 x12 frames, 4 levels, form={form}")
    frames = list(range(0, 100, 8))[:12]
    depths, cam, poses, _ = room_sequence(width=320, height=240, f=262.5, frames=frames)
    cfg = dict(configs.ROOM, form=form, max_blocks=1 << 17, hash_slots=1 << 18)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    merges = 0
    for k in range(len(frames)):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        last, _ = g.sync()
        st = o.integrate_depth(depths[k], cam.K, poses[k])
        assert last["valid_points"] == st["valid_points"]
        assert last["new_blocks"] == st["new_blocks"]
        merges += sum(st["merges"])
    rep = compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"])
    print(rep, "merges", merges)
    assert merges > 100


def _occlusion_frames():
    """A far plane, then occluders in front of it: blocks behind an occluder by more than the
    truncation distance receive no update, also where whole blocks are rejected at once."""
    h, w, f = 120, 160, 150.0
    K = np.array([f, f, w / 2.0, h / 2.0])
    far = np.full((h, w), 2.0, np.float32)
    half = far.copy()
    half[:, : w // 2] = 1.0
    near = np.full((h, w), 1.0, np.float32)
    holes = near.copy()
    holes[30:90, 40:120] = np.nan
    holes[0:20, :] = 0.0
    step = np.where(np.arange(w)[None, :] < w // 3, np.float32(2.07), np.float32(2.0)).repeat(h, 0)
    T = np.eye(4)
    T2 = np.eye(4)
    T2[0, 3] = 0.3  # shifted camera: part of the map leaves the image
    return K, [(far, T), (half, T), (near, T), (holes, T), (step, T), (far, T2), (near, T2)]


@pytest.mark.parametrize("sigma", [0.01, 0.001])
def test_room_merge_thresholds(mrh, orc, sigma):
    """The 4-level room orbit at the other thresholds of the merge sweep (sigma_thr = 10 mm merges
    more blocks than the default 5 mm, 1 mm about a sixth as many): 320x240, 12 frames spread over
    the orbit."""
    announce(f"room 320x240 x12 frames, 4 levels, sigma_thr={sigma}")
    frames = list(range(0, 100, 8))[:12]
    depths, cam, poses, _ = room_sequence(width=320, height=240, f=262.5, frames=frames)
    cfg = dict(configs.ROOM, var_thr=sigma * sigma, max_blocks=1 << 17, hash_slots=1 << 18)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    merges = [0, 0, 0, 0]
    for k in range(len(frames)):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        last, _ = g.sync()
        st = o.integrate_depth(depths[k], cam.K, poses[k])
        assert last["valid_points"] == st["valid_points"]
        assert last["new_blocks"] == st["new_blocks"]
        merges = [a + b for a, b in zip(merges, st["merges"])]
    rep = compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"])
    print(rep, "merges", merges)
    if sigma >= 0.01:
        assert merges[0] > 1000 and merges[1] > 100


@pytest.mark.parametrize("side", [-1, 1])
def test_merge_threshold_closed_form(mrh, orc, side):
    """Two noise-free planes 2 cm apart, seen once each (z-difference form): every voxel seen on
    both frames inside the band has sigma^2 = delta^2 / 4, so the blocks made of such voxels (rows
    z = 11..13 of 16 cm blocks) merge after the second frame with the threshold 1% above that value
    and stay fine 1% below it; the GPU map's levels must equal the oracle's on every block."""
    from workloads import plane_frame

    announce(f"closed-form merge threshold, side {side}")
    d1, cam, T = plane_frame(2.0, 32, 24, 24.0)
    d2, _, _ = plane_frame(2.02, 32, 24, 24.0)
    delta = float(d2[0, 0]) - float(d1[0, 0])
    cfg = dict(voxel=0.02, levels=2, tau=0.3, var_thr=delta * delta / 4.0 * (1.0 + side * 1e-2), max_depth=5.0,
               form="zdiff", max_blocks=1 << 14, hash_slots=1 << 15)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for d in (d1, d2):
        g.integrate_depth(_dev(d), cam.K, T)
        g.sync()
        o.integrate_depth(d, cam.K, T)
    ref = o.extract()
    ex = excused_keys(o)
    assert not any(k[2] in (11, 12, 13) for k in ex)
    print(compare_maps(gpu_sorted(g), ref, excused=ex, tau=cfg["tau"]))
    rows = np.isin(ref.keys[:, 2], [11, 12, 13])
    merged = int((ref.levels[rows] == 1).sum())
    assert (merged >= 8) if side > 0 else (merged == 0), merged


@pytest.mark.parametrize("form", ["range", "zdiff"])
def test_occluded_blocks(mrh, orc, form):
    announce(f"occlusion planes 160x120 x7 frames form={form}")
    K, frames = _occlusion_frames()
    cfg = dict(configs.SPHERE_PLANE, levels=2, var_thr=1e-6, form=form)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k, (d, T) in enumerate(frames):
        g.integrate_depth(_dev(d), K, T)
        last, _ = g.sync()
        st = o.integrate_depth(d, K, T)
        assert last["observations"] == st["observations"], k
        assert last["distinct_voxels"] == st["distinct_voxels"], k
        assert last["candidate_keys"] == st["candidate_keys"], k
        assert last["new_blocks"] == st["new_blocks"], k
    rep = compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"])
    print(rep)


@pytest.mark.parametrize("size", [(203, 157), (17, 1)])
def test_room_ragged_frame_sizes(mrh, orc, size):
    """Frames whose width and height are not multiples of the 16x16 pixel tile (a partial last
    tile row and column, half-pixel principal point), 4 frames of the orbit."""
    w, h = size
    announce(f"room ragged {w}x{h} x4 frames, 4 levels")
    depths, cam, poses, _ = room_sequence(width=w, height=h, f=0.82 * w, frames=[0, 9, 18, 27])
    cfg = dict(configs.ROOM, max_blocks=1 << 16, hash_slots=1 << 17)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k in range(len(depths)):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        last, _ = g.sync()
        st = o.integrate_depth(depths[k], cam.K, poses[k])
        assert last["valid_points"] == st["valid_points"], k
        assert last["new_blocks"] == st["new_blocks"], k
        assert last["observations"] == st["observations"], k
        assert last["distinct_voxels"] == st["distinct_voxels"], k
        assert last["candidate_keys"] == st["candidate_keys"], k
    assert o.num_blocks > 0
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]))


def test_room_full_size_first_frames(mrh, orc):
    """640x480 at the full configuration, first 3 frames; then the benchmark's query launch (1M
    points near the surfaces, the same query pose) on that map, sampled outputs against the
    oracle one by one, and its adjoint over all 1M points against the oracle's."""
    announce("room 640x480 x3 frames full config")
    from workloads import surface_query_points

    depths, cam, poses, scene = room_sequence(frames=[0, 1, 2])
    g = mrh.Map(**configs.ROOM)
    o = orc.OracleMap(**configs.oracle_kwargs(configs.ROOM))
    for k in range(3):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        o.integrate_depth(depths[k], cam.K, poses[k])
    g.sync()
    ex = excused_keys(o)
    print(compare_maps(gpu_sorted(g), o.extract(), excused=ex, tau=configs.ROOM["tau"]))
    announce("room full config: 1M-point query, 10000 sampled against the oracle")
    pts = surface_query_points(scene, 1_000_000, sigma=0.015, seed=100)
    T = np.eye(4)
    T[:3, 3] = [0.01, -0.01, 0.005]
    sdf, valid, _ = g.query(_dev(pts), T=T)
    idx = np.random.default_rng(5).choice(len(pts), 10000, replace=False)
    osdf, ovalid, _ = o.query(pts[idx], T=T)
    # a sample whose 3x3x3 block neighbourhood holds a block merged within rounding of the
    # threshold may legitimately differ
    B = 8 * configs.ROOM["voxel"]
    pw = pts[idx].astype(np.float64) + T[:3, 3]
    kb = np.floor(pw / B).astype(np.int64)
    near = np.array([any((a + dx, b + dy, c + dz) in ex for dx in (-1, 0, 1) for dy in (-1, 0, 1) for dz in (-1, 0, 1))
                     for a, b, c in kb.tolist()], dtype=bool)
    gv = valid.cpu().numpy()[idx]
    ov = ovalid.astype(bool)
    assert np.array_equal(gv[~near], ov[~near])
    ok = gv & ov & ~near
    assert ok.sum() > 1000
    np.testing.assert_allclose(sdf.cpu().numpy()[idx][ok], osdf[ok], atol=1e-5, rtol=0)
    announce("room full config: 1M-point query adjoint against the oracle's, every point")
    # incoming gradient 1 as in the benchmark, 0 next to excused blocks so that both sides leave
    # them out of the pose gradient too
    kb = np.floor((pts.astype(np.float64) + T[:3, 3]) / B).astype(np.int64)
    code = lambda k: ((k[..., 0] + (1 << 20)) << 42) | ((k[..., 1] + (1 << 20)) << 21) | (k[..., 2] + (1 << 20))
    hood = np.array([(a + dx, b + dy, c + dz) for a, b, c in ex for dx in (-1, 0, 1) for dy in (-1, 0, 1)
                     for dz in (-1, 0, 1)], dtype=np.int64).reshape(-1, 3)
    gs = np.where(np.isin(code(kb), code(hood)), 0.0, 1.0).astype(np.float32)
    gp, gpose = g.query_backward(_dev(pts), _dev(gs), T=T)
    ogp, ogpose = o.query_backward(pts, gs.astype(np.float64), T=T)
    np.testing.assert_allclose(gp.cpu().numpy(), ogp, atol=2e-3, rtol=1e-4)
    np.testing.assert_allclose(gpose, ogpose, rtol=1e-4, atol=1e-6 * np.abs(ogpose).max())


def test_street_sequence_multires(mrh, orc):
    """LiDAR carving at reduced size: 16 rings x 512 azimuths, 5 scans."""
    announce("street 16x512 x5 scans carve 4 levels")
    pts, poses, _ = street_sequence(n_scans=200, rings=16, azimuths=512, scans=[0, 1, 2, 3, 4])
    cfg = dict(configs.STREET, max_blocks=1 << 18, hash_slots=1 << 19)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    merges = 0
    for k in range(pts.shape[0]):
        g.integrate_points(_dev(pts[k]), poses[k])
        last, _ = g.sync()
        st = o.integrate_points(pts[k], poses[k])
        assert last["valid_points"] == st["valid_points"]
        assert last["new_blocks"] == st["new_blocks"]
        assert last["observations"] == st["observations"]
        assert last["distinct_voxels"] == st["distinct_voxels"]
        assert last["candidate_keys"] == st["candidate_keys"]
        assert last["queued_blocks"] == st["touched_blocks"]
        merges += sum(st["merges"])
    rep = compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o))
    print(rep, "merges", merges)
    assert merges > 50


def test_street_full_size_first_scans(mrh, orc):
    """LiDAR at the full street configuration (64 rings x 2048 azimuths, 2^21 blocks, 2^22 slots,
    the launch shapes the benchmark times), first 2 scans: per-scan counts and the whole map."""
    announce("street 64x2048 x2 scans full config")
    pts, poses, _ = street_sequence(rings=64, azimuths=2048, scans=[0, 1])
    g = mrh.Map(**configs.STREET)
    o = orc.OracleMap(**configs.oracle_kwargs(configs.STREET))
    for k in range(pts.shape[0]):
        g.integrate_points(_dev(pts[k]), poses[k])
        last, _ = g.sync()
        st = o.integrate_points(pts[k], poses[k])
        assert last["valid_points"] == st["valid_points"]
        assert last["new_blocks"] == st["new_blocks"]
        assert last["observations"] == st["observations"]
        assert last["distinct_voxels"] == st["distinct_voxels"]
        assert last["candidate_keys"] == st["candidate_keys"]
        assert last["queued_blocks"] == st["touched_blocks"]
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o)))


@pytest.mark.timeout(300)
def test_street_full_sequence(mrh, orc):
    """The benchmark's whole LiDAR workload: the 20 scans of 64 x 2048 points at the full street
    configuration, per-scan counts and the final map (about 394k blocks, 900k merges)."""
    announce("street 64x2048 x20 scans full config (benchmark sequence)")
    pts, poses, _ = street_sequence(rings=64, azimuths=2048, scans=range(20))
    g = mrh.Map(**configs.STREET)
    o = orc.OracleMap(**configs.oracle_kwargs(configs.STREET))
    merges = 0
    for k in range(pts.shape[0]):
        g.integrate_points(_dev(pts[k]), poses[k])
        last, _ = g.sync()
        st = o.integrate_points(pts[k], poses[k])
        assert last["valid_points"] == st["valid_points"], k
        assert last["new_blocks"] == st["new_blocks"], k
        assert last["observations"] == st["observations"], k
        assert last["distinct_voxels"] == st["distinct_voxels"], k
        assert last["candidate_keys"] == st["candidate_keys"], k
        assert last["queued_blocks"] == st["touched_blocks"], k
        merges += sum(st["merges"])
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o)), "merges", merges)


def test_street_band_only(mrh, orc):
    announce("street 8x256 band-only (no carving)")
    pts, poses, _ = street_sequence(n_scans=200, rings=8, azimuths=256, scans=[10, 11])
    cfg = dict(configs.STREET, carve=False, max_blocks=1 << 16, hash_slots=1 << 17)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k in range(2):
        g.integrate_points(_dev(pts[k]), poses[k])
        o.integrate_points(pts[k], poses[k])
    g.sync()
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o)))


def _long_ray_scan(seed):
    """Carving rays hundreds of metres long (more blocks than the per-ray block record holds) mixed
    with short ones."""
    rng = np.random.default_rng(seed)
    far = np.array([[600.0, 0.0, 0.0], [-450.0, 380.0, -20.0], [0.3, 700.0, 5.0], [500.0, -500.0, 40.0]])
    near = rng.normal(size=(60, 3)) * 5.0 + np.array([10.0, 0.0, 0.0])
    return np.concatenate([far, near, far * 0.999]).astype(np.float32)


def test_lidar_long_rays(mrh, orc):
    """Blocks past a ray's recorded capacity are walked by the ray's own lane."""
    announce("lidar carving rays up to 900 m (block record overflow)")
    cfg = dict(voxel=0.05, levels=2, tau=0.15, var_thr=0.025 ** 2, min_obs=2, min_range=1.0, max_range=1000.0,
               carve=True, max_blocks=1 << 17, hash_slots=1 << 18)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k in range(2):
        T = np.eye(4)
        T[:3, 3] = [0.1 + 0.37 * k, 0.2, 1.5]
        pts = _long_ray_scan(k)
        g.integrate_points(_dev(pts), T)
        last, _ = g.sync()
        st = o.integrate_points(pts, T)
        assert last["observations"] == st["observations"], k
        assert last["distinct_voxels"] == st["distinct_voxels"], k
        assert last["candidate_keys"] == st["candidate_keys"], k
        assert last["queued_blocks"] == st["touched_blocks"], k
        assert last["new_blocks"] == st["new_blocks"], k
    assert o.num_blocks > 4 * 1100
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]))


def _query_points(n, seed=0):
    rng = np.random.default_rng(seed)
    return np.stack([rng.uniform(-0.45, 0.45, n), rng.uniform(-0.35, 0.35, n),
                     rng.uniform(1.9, 4.1, n)], axis=1).astype(np.float32)


@pytest.mark.parametrize("strict", [False, True])
def test_query_parity(mrh, orc, strict):
    announce(f"query sphere_plane strict={strict}")
    depth, cam, T = sphere_plane_frame(seed=0)
    d2, _, _ = sphere_plane_frame(seed=1)
    g = mrh.Map(**configs.SPHERE_PLANE)
    o = orc.OracleMap(**configs.oracle_kwargs(configs.SPHERE_PLANE))
    for d in (depth, d2):
        g.integrate_depth(_dev(d), cam.K, T)
        o.integrate_depth(d, cam.K, T)
    pts = _query_points(20000)
    Tq = np.eye(4)
    Tq[:3, 3] = [0.003, -0.002, 0.001]
    sdf, valid, grad = g.query(_dev(pts), T=Tq, strict=strict, with_grad=True)
    osdf, ovalid, ograd = o.query(pts, T=Tq, strict=strict)
    valid = valid.cpu().numpy()
    assert np.array_equal(valid, ovalid)
    assert valid.sum() > 1000
    np.testing.assert_allclose(sdf.cpu().numpy()[valid], osdf[valid], atol=1e-5, rtol=0)
    np.testing.assert_allclose(grad.cpu().numpy()[valid], ograd[valid], atol=2e-3, rtol=1e-4)
    assert np.all(sdf.cpu().numpy()[~valid] == 0)


def test_query_multires_parity(mrh, orc):
    announce("query on a merged 4-level room map")
    frames = list(range(0, 100, 10))
    depths, cam, poses, scene = room_sequence(width=320, height=240, f=262.5, frames=frames)
    cfg = dict(configs.ROOM, max_blocks=1 << 17, hash_slots=1 << 18)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k in range(len(frames)):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        o.integrate_depth(depths[k], cam.K, poses[k])
    g.sync()
    ex = excused_keys(o)
    from workloads import surface_query_points

    pts = surface_query_points(scene, 50000, sigma=0.015, seed=3)
    sdf, valid, grad = g.query(_dev(pts), with_grad=True)
    osdf, ovalid, ograd = o.query(pts)
    # points whose 2x2x2 neighbourhood touches an excused block may legitimately differ
    B = 8 * cfg["voxel"]
    near = np.zeros(len(pts), bool)
    if ex:
        kb = np.floor(pts.astype(np.float64) / B).astype(np.int64)
        for dx in (-1, 0, 1):
            for dy in (-1, 0, 1):
                for dz in (-1, 0, 1):
                    near |= np.array([(a + dx, b + dy, c + dz) in ex for a, b, c in kb.tolist()])
    valid = valid.cpu().numpy()
    assert np.array_equal(valid[~near], ovalid[~near])
    ok = valid & ovalid & ~near
    assert ok.sum() > 10000
    np.testing.assert_allclose(sdf.cpu().numpy()[ok], osdf[ok], atol=1e-5, rtol=0)
    print("levels", np.bincount(o.extract().levels), "excused", len(ex))


def test_query_backward_parity(mrh, orc):
    announce("query backward sphere_plane")
    depth, cam, T = sphere_plane_frame(seed=0)
    g = mrh.Map(**configs.SPHERE_PLANE)
    o = orc.OracleMap(**configs.oracle_kwargs(configs.SPHERE_PLANE))
    g.integrate_depth(_dev(depth), cam.K, T)
    o.integrate_depth(depth, cam.K, T)
    pts = _query_points(30000, seed=5)
    th = np.deg2rad(2.0)
    Tq = np.eye(4)
    Tq[:3, :3] = [[np.cos(th), -np.sin(th), 0], [np.sin(th), np.cos(th), 0], [0, 0, 1]]
    Tq[:3, 3] = [0.05, -0.02, 0.01]
    gs = np.random.default_rng(1).normal(size=len(pts)).astype(np.float32)
    gp, gpose = g.query_backward(_dev(pts), _dev(gs), T=Tq)
    ogp, ogpose = o.query_backward(pts, gs.astype(np.float64), T=Tq)
    np.testing.assert_allclose(gp.cpu().numpy(), ogp, atol=2e-3, rtol=1e-4)
    np.testing.assert_allclose(gpose, ogpose, rtol=1e-4, atol=1e-6 * np.abs(ogpose).max())


def test_sdfquery_autograd(mrh):
    announce("SdfQuery autograd")
    depth, cam, T = sphere_plane_frame(seed=0)
    g = mrh.Map(**configs.SPHERE_PLANE)
    g.integrate_depth(_dev(depth), cam.K, T)
    pts = _dev(_query_points(4000, seed=7)).requires_grad_(True)
    sdf, valid = mrh.SdfQuery.apply(g, pts)
    (sdf * valid.float()).sum().backward()
    ref, rvalid, rgrad = g.query(pts.detach().contiguous(), with_grad=True)
    np.testing.assert_allclose(pts.grad.cpu().numpy()[rvalid.cpu().numpy()],
                               rgrad.cpu().numpy()[rvalid.cpu().numpy()], rtol=1e-6, atol=1e-6)
    assert g.last_pose_grad.shape == (6,)


def test_empty_and_invalid_inputs(mrh):
    announce("empty / invalid inputs")
    g = mrh.Map(**configs.SPHERE_PLANE)
    depth = torch.full((240, 320), float("nan"), device="cuda")
    depth[0, :10] = -1.0
    depth[1, :10] = 0.0
    depth[2, :10] = float("inf")
    K = [300.0, 300.0, 160.0, 120.0]
    g.integrate_depth(depth, K, np.eye(4))
    last, tot = g.sync()
    assert last["valid_points"] == 0 and last["new_blocks"] == 0 and tot["blocks"] == 0
    g.integrate_points(torch.zeros((0, 3), device="cuda"), np.eye(4))
    g.sync()
    with pytest.raises(mrh.MrhError):
        g.integrate_depth(depth, K, np.full((4, 4), np.nan))
    with pytest.raises(mrh.MrhError):
        g.integrate_depth(depth, [0.0, 300.0, 160.0, 120.0], np.eye(4))
    assert g.counts() == (0, 0)


def test_capacity_errors(mrh, orc):
    announce("table / heap / block capacity errors")
    depth, cam, T = sphere_plane_frame(seed=0)
    d = _dev(depth)
    g = mrh.Map(**dict(configs.SPHERE_PLANE, max_blocks=512, hash_slots=4096, heap_blocks=[4096, 0, 0, 0]))
    g.integrate_depth(d, cam.K, T)
    with pytest.raises(mrh.MrhError) as ei:
        g.sync()
    assert ei.value.code == -7  # block limit (1184 blocks > 512)
    h = mrh.Map(**dict(configs.SPHERE_PLANE, heap_blocks=[100, 0, 0, 0]))
    h.integrate_depth(d, cam.K, T)
    with pytest.raises(mrh.MrhError) as ei:
        h.sync()
    assert ei.value.code == -4  # heap full
    nb, nv = h.counts()
    assert nv == 100 * 512  # blocks without storage report no voxels
    # a probe limit of one slot: any two of the frame's keys sharing an Eq. 4 home slot make the
    # second insert fail; the host evaluation of the hash shows such a pair exists
    slots = 4096
    o = orc.OracleMap(**configs.oracle_kwargs(configs.SPHERE_PLANE))
    o.integrate_depth(depth, cam.K, T)
    homes = [mrh.block_hash(int(x), int(y), int(z), slots) for x, y, z in o.extract().keys.tolist()]
    collide = len(homes) - len(set(homes))
    assert collide > 0
    t = mrh.Map(**dict(configs.SPHERE_PLANE, max_blocks=2048, hash_slots=slots, max_probe=1))
    t.integrate_depth(d, cam.K, T)
    with pytest.raises(mrh.MrhError) as ei:
        t.sync()
    assert ei.value.code == -3  # table full
    _, tot = t.sync()  # the latch was cleared by the failing sync; totals still count the losses
    assert tot["failed_inserts"] >= collide


def test_reset_reuses_map(mrh, orc):
    announce("reset and refuse")
    depth, cam, T = sphere_plane_frame(seed=0)
    g = mrh.Map(**configs.SPHERE_PLANE)
    for _ in range(2):
        g.integrate_depth(_dev(depth), cam.K, T)
        g.reset()
    g.integrate_depth(_dev(depth), cam.K, T)
    g.sync()
    o = orc.OracleMap(**configs.oracle_kwargs(configs.SPHERE_PLANE))
    o.integrate_depth(depth, cam.K, T)
    compare_maps(gpu_sorted(g), o.extract(), tau=0.06)


def test_table_full_before_block_limit(mrh):
    """1184 distinct blocks cannot fit a 1024-slot table: the insert reports a full table."""
    announce("table full")
    depth, cam, T = sphere_plane_frame(seed=0)
    g = mrh.Map(**dict(configs.SPHERE_PLANE, max_blocks=512, hash_slots=1024))
    g.integrate_depth(_dev(depth), cam.K, T)
    with pytest.raises(mrh.MrhError) as ei:
        g.sync()
    assert ei.value.code == -3
    nb, _ = g.counts()
    assert nb == 512


def test_sequence_entry_points_equal_frame_calls(mrh):
    """The library-side frame loop gives the same map as one call per frame."""
    announce("sequence entry points")
    depths, cam, poses, _ = room_sequence(width=320, height=240, f=262.5, frames=[0, 5, 10, 15])
    cfg = dict(configs.ROOM, max_blocks=1 << 16, hash_slots=1 << 17)
    a, b = mrh.Map(**cfg), mrh.Map(**cfg)
    d = _dev(depths)
    for k in range(4):
        a.integrate_depth(d[k], cam.K, poses[k])
    b.integrate_depth_sequence(d, cam.K, np.ascontiguousarray(poses))
    ga, gb = gpu_sorted(a), gpu_sorted(b)
    assert np.array_equal(ga.keys, gb.keys) and np.array_equal(ga.D, gb.D) and np.array_equal(ga.W, gb.W)
    pts, sposes, _ = street_sequence(rings=8, azimuths=256, scans=[0, 1, 2])
    cfgs = dict(configs.STREET, max_blocks=1 << 16, hash_slots=1 << 17)
    c, e = mrh.Map(**cfgs), mrh.Map(**cfgs)
    x = _dev(pts)
    for k in range(3):
        c.integrate_points(x[k], sposes[k])
    e.integrate_points_sequence(x, np.ascontiguousarray(sposes))
    gc, ge = gpu_sorted(c), gpu_sorted(e)
    assert np.array_equal(gc.keys, ge.keys) and np.array_equal(gc.D, ge.D) and np.array_equal(gc.W, ge.W)


@pytest.mark.parametrize("form", ["range", "zdiff"])
@pytest.mark.parametrize("shift", [0.5, 0.5 - 2.0 ** -40, 0.25])
def test_pixel_boundaries(mrh, orc, form, shift):
    """Voxel centres that project exactly on pixel boundaries (dyadic sizes and pose), next to them by less
    than the fast projection's margin, and off them: every decision is the canonical one."""
    announce(f"pixel boundaries {form} shift {shift}")
    cfg = dict(voxel=1.0 / 32, levels=2, tau=3.0 / 32, var_thr=1e-6, min_obs=2, max_depth=5.0, form=form,
               max_blocks=1 << 13, hash_slots=1 << 14)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    K = (32.0, 32.0, 15.5, 11.5)
    T = np.eye(4)
    T[:3, 3] = shift / 32
    rng = np.random.default_rng(5)
    depth = np.where(rng.random((24, 32)) < 0.5, 1.0, 2.0).astype(np.float32)
    depth[3:6, 4:9] = 0.0
    for k in range(3):
        g.integrate_depth(_dev(depth), K, T)
        last, _ = g.sync()
        st = o.integrate_depth(depth, K, T)
        for a in ("valid_points", "new_blocks", "observations", "distinct_voxels", "candidate_keys"):
            assert last[a] == st[a], (k, a)
    assert o.num_blocks > 50
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]))


@pytest.mark.parametrize("size", [((1 << 23) + 1, 2), ((1 << 24) - 1, 2), (2, (1 << 23) + 300)])
def test_sides_from_2_to_the_23(mrh, orc, size):
    """Frames with a side of 2^23 pixels and more (sides below 2^24 are accepted): valid depths in 140 pixels
    near the far end of the long side, in both lines of the short one."""
    w, h = size
    announce(f"flat frame {w}x{h} x2")
    cfg = dict(voxel=0.005, levels=3, tau=0.02, var_thr=0.004 ** 2, min_obs=2, max_depth=5.0, max_blocks=1 << 14,
               hash_slots=1 << 15)
    depth = np.zeros((h, w), np.float32)
    rng = np.random.default_rng(4)
    long = max(w, h)
    sel = np.s_[:, long - 160:long - 20] if w > h else np.s_[long - 160:long - 20, :]
    depth[sel] = rng.uniform(0.98, 1.02, depth[sel].shape)
    K = (100.0, 100.0, long - 90.0 if w > h else 0.5, 0.5 if w > h else long - 90.0)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    dev = _dev(depth)
    for k in range(2):
        g.integrate_depth(dev, K, np.eye(4))
        last, _ = g.sync()
        st = o.integrate_depth(depth, K, np.eye(4))
        for a in ("valid_points", "new_blocks", "observations", "distinct_voxels", "candidate_keys"):
            assert last[a] == st[a], (k, a)
    assert st["valid_points"] == 280 and st["observations"] > 10000
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]))


@pytest.mark.parametrize("form", ["range", "zdiff"])
def test_max_depth_nan_takes_no_sample(mrh, form):
    """No depth is <= a maximum depth that is not a number: a frame changes nothing, also not the blocks
    that are there."""
    announce(f"maximum depth NaN, {form}")
    g = mrh.Map(voxel=0.05, levels=4, tau=0.15, max_depth=float("nan"), form=form, max_blocks=64)
    keys = np.array([[0, 0, 2], [-1, 0, 2], [0, -1, 2], [-1, -1, 2]], np.int32)
    nv = 512 + 64 + 8 + 1
    assert g.load_blocks(keys, np.arange(4), np.full(nv, 0.1, np.float32), np.full(nv, 3, np.uint32), np.zeros(nv, np.float32)) == 4
    before = gpu_sorted(g)
    g.integrate_depth(torch.full((48, 64), 0.9, device="cuda"), [60.0, 60.0, 31.5, 23.5], np.eye(4))
    last, _ = g.sync()
    assert last["valid_points"] == last["observations"] == last["new_blocks"] == 0
    after = gpu_sorted(g)
    for a in ("keys", "levels", "D", "W", "S2"):
        assert np.array_equal(getattr(before, a), getattr(after, a)), a
