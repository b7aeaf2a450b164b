"""LiDAR fusion and queries where their kernels split the work: rays along and exactly on the block
lattice, scans at the edges of a workgroup's rays, scans whose band counts need words of their own,
queries and frames at the edges of a workgroup.  Against the oracle, exactly for counts and
discrete decisions (both sides decide them in FP64 by the same expressions)."""
import numpy as np
import pytest
import torch

from parity_util import announce, compare_maps, excused_keys, gpu_sorted
from workloads import configs, room_sequence

pytestmark = pytest.mark.gpu

CFG = dict(voxel=0.05, levels=4, tau=0.15, var_thr=0.025 ** 2, min_obs=2, min_range=0.5, max_range=80.0, carve=True,
           max_blocks=1 << 16, hash_slots=1 << 17)


@pytest.fixture(scope="module")
def mrh():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2511_21459_amd as mrh

    return mrh


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _scans_match(mrh, orc, cfg, scans):
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    merges = 0
    for k, (pts, T) in enumerate(scans):
        g.integrate_points(_dev(pts), T)
        last, _ = g.sync()
        st = o.integrate_points(pts, T)
        for a, b in (("valid_points", "valid_points"), ("new_blocks", "new_blocks"), ("observations", "observations"),
                     ("distinct_voxels", "distinct_voxels"), ("candidate_keys", "candidate_keys"),
                     ("queued_blocks", "touched_blocks")):
            assert last[a] == st[b], (k, a)
        merges += sum(st["merges"])
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]), "merges", merges)
    return merges


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 129])
@pytest.mark.parametrize("origin", [0.0, 0.4, 0.025])
def test_rays_on_the_lattice(mrh, orc, n, origin):
    """Axis-parallel and diagonal rays from an origin on a block corner (0, 0.4: ties on every step) and
    on a voxel centre, with ends on corners and off them; four scans, so that blocks merge."""
    announce(f"lattice rays n={n} origin={origin}")
    dirs = np.array([[1, 0, 0], [0, -1, 0], [0, 0, 1], [1, 1, 0], [-1, 0, 1], [0, 1, -1], [1, 1, 1], [-1, -1, 1], [1, -2, 3],
                     [0.3, 0.7, -0.2], [-1, 0, 0], [0, 1, 0], [0, 0, -1]])
    reach = np.array([0.8, 1.2, 2.0, 4.4, 0.9375, 3.1])
    k = np.arange(n)
    pts = (dirs[k % len(dirs)] * reach[k // 3 % len(reach)][:, None]).astype(np.float32)
    T = np.eye(4)
    T[:3, 3] = origin
    _scans_match(mrh, orc, CFG, [(pts, T)] * 4)


@pytest.mark.parametrize("n", [0, 1, 255, 4099, 16385])
def test_scan_sizes(mrh, orc, n):
    """Scans in general position of few and many rays, the table and touched lists of their workgroups
    full and nearly empty; moving, so that new, merging and merged blocks are updated together."""
    announce(f"scan of {n} rays")
    rng = np.random.default_rng(n)
    d = rng.normal(size=(n, 3))
    pts = (d / np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-9) * rng.uniform(1.0, 12.0, (n, 1))).astype(np.float32)
    scans = []
    for k in range(5):
        T = np.eye(4)
        T[:3, 3] = [0.03 + 0.11 * k, 0.02, -0.01]
        scans.append((pts, T))
    merges = _scans_match(mrh, orc, dict(CFG, max_blocks=1 << 18, hash_slots=1 << 19), scans)
    assert n < 1000 or merges > 50


def test_counts_apart(mrh, orc):
    """A scan whose sums could outgrow the word they share with the count (rays x truncation), between
    scans that fit it, on one map."""
    announce("wide band counts")
    cfg = dict(CFG, voxel=0.5, tau=4.0, min_range=1.0, max_range=400.0, var_thr=0.01, carve=False)
    rng = np.random.default_rng(3)
    scans = []
    for k, n in enumerate((500, 140000, 700)):  # 140000 x 2 x 4 m x 2^24 > 2^44
        d = rng.normal(size=(n, 3))
        pts = (d / np.linalg.norm(d, axis=1, keepdims=True) * rng.uniform(20.0, 30.0, (n, 1))).astype(np.float32)
        T = np.eye(4)
        T[:3, 3] = [0.1, 0.2 * k, 0.3]
        scans.append((pts, T))
    _scans_match(mrh, orc, cfg, scans)


@pytest.mark.parametrize("size", [(1, 1), (16, 16), (17, 33)])
def test_frames_of_few_workgroups(mrh, orc, size):
    """Frames of one and a few tiles: the hand-off between frames is shared by few workgroups."""
    w, h = size
    announce(f"room {w}x{h} x6 frames")
    depths, cam, poses, _ = room_sequence(width=w, height=h, f=0.82 * w, frames=[0, 1, 2, 3, 4, 5])
    cfg = dict(configs.ROOM, max_blocks=1 << 14, hash_slots=1 << 15)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    for k in range(len(depths)):
        g.integrate_depth(_dev(depths[k]), cam.K, poses[k])
        last, _ = g.sync()
        st = o.integrate_depth(depths[k], cam.K, poses[k])
        for a in ("valid_points", "new_blocks", "observations", "distinct_voxels", "candidate_keys"):
            assert last[a] == st[a], (k, a)
    print(compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"]))


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("strict", [False, True])
def test_query_group_edges(mrh, storage, strict):
    """Queries of n points equal the first n of a long one, for n at the edges of a workgroup's 64 points."""
    announce(f"query edges {storage} strict={strict}")
    depths, cam, poses, _ = room_sequence(width=160, height=120, f=131.0, frames=[0, 5, 10, 15])
    m = mrh.Map(**dict(configs.ROOM, max_blocks=1 << 15, hash_slots=1 << 16, storage=storage))
    for k in range(len(depths)):
        m.integrate_depth(_dev(depths[k]), cam.K, poses[k])
    e = m.extract(voxels=False)
    keys = e["keys"].cpu().numpy()
    rng = np.random.default_rng(2)
    pts = _dev(((keys[rng.integers(0, len(keys), 700)] + rng.random((700, 3))) * 8 * configs.ROOM["voxel"]).astype(np.float32))
    T = np.eye(4)
    T[:3, 3] = [0.003, -0.002, 0.001]
    for grad in (False, True):
        full = m.query(pts, T=T, strict=strict, with_grad=grad)
        assert 20 < int(full[1].sum()) < 700
        for n in (0, 1, 63, 64, 65, 129):
            part = m.query(pts[:n].contiguous(), T=T, strict=strict, with_grad=grad)
            for a, b in zip(part, full):
                if a is not None:
                    assert torch.equal(a, b[:n]), (n, grad)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("strict", [False, True])
def test_query_large_batches(mrh, storage, strict):
    """A query of many points gives each what queries of few give it, at the sizes where the lookup of 64 points per
    wave begins and ends, with waves whose points all have a block, some, one or none; the adjoint's pose gradient is
    the same sum in another order (FP64, 6e5 terms: 1e-9 of the terms' absolute sum is far above its rounding)."""
    announce(f"large query batches {storage} strict={strict}")
    depths, cam, poses, _ = room_sequence(width=160, height=120, f=131.0, frames=[0, 5, 10, 15])
    m = mrh.Map(**dict(configs.ROOM, max_blocks=1 << 15, hash_slots=1 << 16, storage=storage))
    for k in range(len(depths)):
        m.integrate_depth(_dev(depths[k]), cam.K, poses[k])
    keys = m.extract(voxels=False)["keys"].cpu().numpy()
    rng = np.random.default_rng(4)
    size = (1 << 19) + 70001
    pts = (keys[rng.integers(0, len(keys), size)] + rng.random((size, 3))) * 8 * configs.ROOM["voxel"]
    share = np.repeat(rng.choice([0.0, 0.02, 0.5, 1.0], size // 64 + 1), 64)[:size]
    pts[rng.random(size) < share] += 500.0
    far = rng.integers(0, size, 50)
    pts[far] = rng.choice([1e30, -3e7, 3e38], (50, 3))
    pts, up = _dev(pts.astype(np.float32)), _dev(rng.standard_normal(size).astype(np.float32))
    T = np.eye(4)
    T[:2, :2] = [[0.8, -0.6], [0.6, 0.8]]
    few = 100000
    parts = [slice(a, min(a + few, size)) for a in range(0, size, few)]
    for pose in (None, T):
        apart = [m.query(pts[s].contiguous(), T=pose, strict=strict, with_grad=True) for s in parts]
        want = [torch.cat(c) for c in zip(*apart)]
        assert want[1].any() and not want[1].all()
        for n in ((1 << 19) - 1, 1 << 19, (1 << 19) + 1, (1 << 19) + 65, size):
            for grad in (False, True):
                got = m.query(pts[:n].contiguous(), T=pose, strict=strict, with_grad=grad)
                for a, b in zip(got, want):
                    assert a is None or torch.equal(a, b[:n]), (n, grad)
        gp, pg = [], []
        for s in parts:
            g, p6 = m.query_backward(pts[s].contiguous(), up[s].contiguous(), T=pose, strict=strict)
            gp.append(g)
            pg.append(np.asarray(p6))
        gp = torch.cat(gp)
        bound = float((gp.double().abs().sum(dim=1) * (1.0 + 2.0 * pts.double().abs().sum(dim=1))).sum())
        g, p6 = m.query_backward(pts, up, T=pose, strict=strict)
        assert torch.equal(g, gp)
        assert np.abs(np.asarray(p6) - sum(pg)).max() <= 1e-9 * bound
        # a point that is not finite: the pose terms that it enters by x cross dL/dx are NaN, as in small batches
        odd = pts.clone()
        for rows, value in ((slice(300, 301), (1.0, float("nan"), 2.0)), (slice(size - 1, size), (-float("inf"), 1.0, 2.0))):
            odd[rows] = torch.tensor(value, device=odd.device)
            for b, s in ((odd, slice(0, size)), (odd, slice(max(0, rows.start - 200), rows.stop))):
                got = m.query(b[s].contiguous(), T=None, strict=strict)
                assert not got[1][rows.start - s.start] and got[0][rows.start - s.start] == 0
                bad = np.isnan(m.query_backward(b[s].contiguous(), up[s].contiguous(), T=None, strict=strict)[1])
                axes = ~np.isfinite(odd[s].cpu().numpy()).all(axis=0)
                assert list(bad) == [False] * 3 + [bool(axes[(k + 1) % 3] or axes[(k + 2) % 3]) for k in range(3)]
        for n in ((1 << 17) - 1, 1 << 17, (1 << 17) + 1):
            assert torch.equal(m.query_backward(pts[:n].contiguous(), up[:n].contiguous(), T=pose, strict=strict)[0], gp[:n]), n


def _one_line(rng, n, lo, hi):
    """n points along one direction: every ray crosses the same voxels."""
    d = np.array([0.48, 0.6, 0.64])
    return (d * rng.uniform(lo, hi, (n, 1))).astype(np.float32)


@pytest.mark.parametrize("n", [20000, 140000])
def test_squares_apart(mrh, orc, n):
    """A scan whose observations of one voxel have squares that sum to more than 2^16 m^2 (what 64 bits hold
    in units of 2^-48 m^2), with counts beside the sums (20000 rays) and apart (140000), between scans that
    stay below it, on one map."""
    announce(f"wide sums of squares, {n} rays through the same voxels")
    cfg = dict(CFG, voxel=0.5, tau=4.0, min_range=1.0, max_range=400.0, var_thr=0.01, carve=False)
    rng = np.random.default_rng(n)
    T = np.eye(4)
    T[:3, 3] = [0.1, 0.2, 0.3]
    _scans_match(mrh, orc, cfg, [(_one_line(rng, k, 19.0, 21.0), T) for k in (500, n, 700)])


def test_more_rays_than_the_shared_count(mrh, orc):
    """2^20 and more observations of one voxel in one scan."""
    n = (1 << 20) + 40000
    announce(f"{n} rays through the same voxels")
    rng = np.random.default_rng(8)
    T = np.eye(4)
    T[:3, 3] = [0.01, 0.02, 0.03]
    _scans_match(mrh, orc, dict(CFG, carve=False), [(_one_line(rng, k, 4.0, 4.1), T) for k in (300, n, 400)])


@pytest.mark.parametrize("n", [1, 2, 4])
def test_failed_inserts_count_keys(mrh, orc, n):
    """Inserts lost to a full table are counted once for the rays of a wave that ask for the same key: with a
    probe limit of one slot, the keys of a ray that find their home slot taken, however many rays walk along
    with it."""
    announce(f"full table, {n} rays")
    cfg = dict(CFG, max_blocks=16, hash_slots=32, max_probe=1)
    pts = np.repeat(np.array([[1.9, 1.3, 0.7]], np.float32), n, 0)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    o.integrate_points(pts, np.eye(4))
    homes = [mrh.block_hash(*map(int, k), 32) for k in o.extract().keys]
    assert len(homes) <= 12 and len(set(homes)) < len(homes)
    g = mrh.Map(**cfg)
    g.integrate_points(_dev(pts), np.eye(4))
    with pytest.raises(mrh.MrhError) as ei:
        g.sync()
    assert ei.value.code == -3
    _, tot = g.sync()
    assert tot["new_blocks"] == len(set(homes))
    assert tot["failed_inserts"] == len(homes) - len(set(homes))


def test_refused_scan_leaves_the_map_usable(mrh, orc):
    """A scan whose ray buffers no GPU holds is refused for lack of memory before it reads anything; the map
    goes on as if it had not been called."""
    import ctypes

    announce("oversized scan refused")
    rng = np.random.default_rng(6)
    d = rng.normal(size=(3000, 3))
    pts = (d / np.linalg.norm(d, axis=1, keepdims=True) * rng.uniform(1.0, 8.0, (3000, 1))).astype(np.float32)
    cfg = dict(CFG, max_blocks=1 << 16, hash_slots=1 << 17)
    g = mrh.Map(**cfg)
    o = orc.OracleMap(**configs.oracle_kwargs(cfg))
    dev, T = _dev(pts), np.eye(4)
    for k in range(3):
        st = mrh._lib.load().mrh_integrate_points(g._h, ctypes.c_void_p(dev.data_ptr()), ctypes.c_int64(1 << 33),
                                                  T.ctypes.data_as(ctypes.c_void_p))
        assert st == -2 and "memory" in mrh._lib.load().mrh_last_error(g._h).decode()
        g.integrate_points(dev, T)
        last, _ = g.sync()
        assert last["observations"] == o.integrate_points(pts, T)["observations"]
    compare_maps(gpu_sorted(g), o.extract(), excused=excused_keys(o), tau=cfg["tau"])


@pytest.mark.parametrize("n", [2560, 2561, 5121, 10241])
def test_blocks_per_task(mrh, orc, n):
    """Scans that touch n blocks each, on both sides of the counts at which an update task takes more blocks: a
    point in the middle of each, without carving; four scans, so that half of the blocks merge."""
    announce(f"{n} blocks per scan")
    cfg = dict(CFG, carve=False, var_thr=0.02 ** 2, max_blocks=1 << 15, hash_slots=1 << 16)
    k = np.arange(n)
    keys = np.stack([k % 25 - 12, k // 25 % 25 - 12, 4 + k // 625], 1)
    rng = np.random.default_rng(n)
    T = np.eye(4)
    scans = []
    for _ in range(4):
        far = rng.normal(0.0, np.where(k % 2 == 0, 0.001, 0.05))  # along the ray: small and large variances
        p = (keys + 0.5) * 0.4
        scans.append(((p * (1.0 + np.clip(far, -0.05, 0.05) / np.linalg.norm(p, axis=1))[:, None]).astype(np.float32), T))
    assert _scans_match(mrh, orc, cfg, scans) > n // 4
