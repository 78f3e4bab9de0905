"""GPU parity of the Monotone Scene Generation tree (readings M1-M5 of the
oracle source; the variant 2.0-B, Sec. III-B and Sec. VI-A) against the
oracle.

Edges: monotonicity, |dR \\ C| and the observed points charged are integer
results and must agree exactly, as must J_r and J_o without colour; with
colour the counts may differ by the binary32 colour decisions, within
ceil(0.001 L) for J_r and ceil(0.001 Q) + ceil(0.001 L) for J_o.  Searches
(integer costs without colour) must return the same goal and score the same
number of successors.
"""
import math
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2008_00326_amd as pk  # noqa: E402
from paper_2008_00326_amd.workloads import make_config  # noqa: E402
from test_oracle_msg import DELTA, _world  # noqa: E402

THREADS = 16


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pk.Context(0)
    yield c
    c.close()


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def check_edges(got, exp, rgb, what):
    v, jr, jo, nr, nq = [t.cpu().numpy() for t in got]
    ev, ejr, ejo, enr, enq = exp
    assert np.array_equal(v, ev), f"{what}: monotone flags differ at {np.flatnonzero(v != ev)[:8]}"
    assert np.array_equal(nr, enr), f"{what}: |dR \\ C| differs at {np.flatnonzero(nr != enr)[:8]}"
    assert np.array_equal(nq, enq), f"{what}: charged points differ at {np.flatnonzero(nq != enq)[:8]}"
    if not rgb:
        assert np.array_equal(jr, ejr), f"{what}: J_r differs at {np.flatnonzero(jr != ejr)[:8]}"
        assert np.array_equal(jo, ejo), f"{what}: J_o differs at {np.flatnonzero(jo != ejo)[:8]}"
        return
    tl = np.array([math.ceil(0.001 * x) for x in enr])
    tq = np.array([math.ceil(0.001 * x) for x in enq])
    assert np.all(np.abs(jr - ejr) <= tl), f"{what}: J_r beyond tolerance"
    assert np.all(np.abs(jo - ejo) <= tq + tl), f"{what}: J_o beyond tolerance"


FLAGS = [oracle.MARK_OCCLUDERS, oracle.MARK_OCCLUDERS | oracle.USE_RGB, oracle.MARK_OCCLUDERS | oracle.VOL_LABEL,
         oracle.VOL_CYL | oracle.USE_RGB, oracle.VOL_LABEL | oracle.USE_RGB]
STATES = [(), ((0, 0),), ((0, 0), (1, 1)), ((2, 1), (0, 3)), ((1, 2),), ((0, 2), (2, 3))]


@pytest.mark.parametrize("flags", FLAGS)
@pytest.mark.parametrize("stride", [1, 2])
def test_edges_match_oracle(ctx, flags, stride):
    meshes, scene, gt, cands = _world(seed=3)
    rgb = bool(flags & oracle.USE_RGB)
    say(f"msg edges: flags {flags}, stride {stride}")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, scene.labels, delta_mm=DELTA, tau_c=20.0, flags=flags,
                        stride=stride)
    mids = [ctx.load_mesh(m.xyz, m.tri, m.rgb) for m in meshes]
    tc = [_cuda(c) for c in cands]
    torch.cuda.synchronize()
    say("  scene and meshes resident")
    checked = 0
    for seq in STATES:
        placed = {o for o, _ in seq}
        ostate = [(meshes[o], o + 1, cands[o][k]) for o, k in seq]
        # only monotone states can be composed
        ok = True
        for n, (o, k) in enumerate(seq):
            v = oracle.msg_expand(scene, ostate[:n], meshes[o], cands[o][k:k + 1], label=o + 1, delta_mm=DELTA,
                                  tau_c=20.0, flags=flags, stride=stride)[0]
            ok &= bool(v[0])
            if not ok:
                break
        if not ok:
            continue
        gstate = [(mids[o], o + 1, cands[o][k]) for o, k in seq]
        for o in range(3):
            if o in placed:
                continue
            say(f"  state {seq}, object {o}: GPU edges")
            got = ctx.msg_expand(sid, gstate, mids[o], tc[o], label=o + 1)
            torch.cuda.synchronize()
            say("  oracle edges")
            exp = oracle.msg_expand(scene, ostate, meshes[o], cands[o], label=o + 1, delta_mm=DELTA, tau_c=20.0,
                                    flags=flags, stride=stride, threads=THREADS)
            check_edges(got, exp, rgb, f"state {seq} object {o}")
            checked += 1
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    assert checked >= 8


@pytest.mark.parametrize("beam", [0, 1, 4])
@pytest.mark.parametrize("flags", [oracle.MARK_OCCLUDERS, oracle.VOL_LABEL])
def test_search_matches_oracle(ctx, beam, flags):
    meshes, scene, gt, cands = _world(seed=5, colours=False)
    rng = np.random.default_rng(6)
    depth = scene.depth.astype(np.int32)
    noisy = np.where(depth > 0, np.clip(depth + np.rint(rng.normal(0, 2.0, depth.shape)), 1, 65534), 0)
    scene.depth = noisy.astype(np.uint16)
    say(f"msg search: beam {beam}, flags {flags}")
    sid = ctx.set_scene(scene.K, scene.depth, None, scene.labels, delta_mm=DELTA, flags=flags)
    mids = [ctx.load_mesh(m.xyz, m.tri, None) for m in meshes]
    objs = [(mids[o], o + 1, _cuda(cands[o])) for o in range(3)]
    got = ctx.msg_search(sid, objs, beam=beam)
    say(f"  GPU search done: {got}")
    exp = oracle.msg_search(scene, [(meshes[o], o + 1, cands[o]) for o in range(3)], beam=beam, delta_mm=DELTA,
                            flags=flags, threads=THREADS)
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    assert got == exp, (got, exp)


@pytest.mark.parametrize("flags", [oracle.MARK_OCCLUDERS, oracle.USE_RGB | oracle.VOL_LABEL])
@pytest.mark.parametrize("delta", [1.5, 60.0])
def test_search_windows_of_one_tile_and_of_several_blocks(ctx, flags, delta):
    """J_o windows within a 4x4 pixel tile, and over more than 8x8 of them
    (delta 60 mm at 0.8 m and f = 300: some 49 pixels), from the root and
    from a state whose points compete with the successor's own."""
    meshes, scene, gt, cands = _world(seed=3)
    rgb = bool(flags & oracle.USE_RGB)
    kw = dict(delta_mm=delta, tau_c=20.0, flags=flags)
    say(f"msg windows: flags {flags}, delta {delta}")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, scene.labels, **kw)
    mids = [ctx.load_mesh(m.xyz, m.tri, m.rgb) for m in meshes]
    checked = 0
    for seq in ((), ((0, 0),), ((2, 1),)):
        ostate = [(meshes[o], o + 1, cands[o][k]) for o, k in seq]
        gstate = [(mids[o], o + 1, cands[o][k]) for o, k in seq]
        for o in {0, 1, 2} - {o for o, _ in seq}:
            got = ctx.msg_expand(sid, gstate, mids[o], _cuda(cands[o]), label=o + 1)
            exp = oracle.msg_expand(scene, ostate, meshes[o], cands[o], label=o + 1, threads=THREADS, **kw)
            check_edges(got, exp, rgb, f"delta {delta} state {seq} object {o}")
            checked += int(exp[0].sum())
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    assert checked >= 8


def _random_world(seed):
    """Three boxes of random sizes at random nearby table positions and yaws
    (some touching or hiding one another), each with four random candidates
    around its generating pose."""
    from paper_2008_00326_amd.workloads.scenes import camera_rig, table_pose
    from test_oracle_msg import _compose
    from tiny_meshes import TScene, box
    rng = np.random.default_rng(900 + seed)
    rig = camera_rig(float(rng.uniform(650, 950)), float(rng.uniform(35, 60)))
    meshes, gt, cands, placed = [], [], [], []
    for k in range(3):
        half = rng.uniform(15, 40, 2)
        meshes.append(box((-half[0], -half[1], 0), (half[0], half[1], rng.uniform(30, 90)), n=int(rng.integers(2, 4)),
                          rgb_seed=int(rng.integers(1 << 30))))
        rad = float(np.hypot(*half))
        while True:            # footprints may touch but hardly interpenetrate
            x, y = rng.uniform(-90, 90, 2)
            if all(np.hypot(x - px, y - py) >= 0.85 * (rad + pr) for px, py, pr in placed):
                break
        placed.append((x, y, rad))
        a = rng.uniform(0, 6.28)
        gt.append(table_pose(rig, x, y, a).reshape(12).astype(np.float32))
        cands.append(np.stack([table_pose(rig, x + dx, y + dy, a + da).reshape(12).astype(np.float32)
                               for dx, dy, da in [(0, 0, 0)] + [tuple(rng.normal(0, [12, 12, 0.25])) for _ in range(3)]]))
    depth, rgb, own = _compose(meshes, gt)
    noisy = np.where(depth > 0, np.clip(depth.astype(np.int32) + np.rint(rng.normal(0, 1.5, depth.shape)), 1, 65534), 0)
    return meshes, TScene((160, 120, 300.0, 300.0, 80.0, 60.0), noisy.astype(np.uint16), rgb, own + 1), gt, cands


@pytest.mark.parametrize("seed", range(8))
def test_random_worlds_match_oracle(ctx, seed):
    """Random worlds, flags, strides and deltas: every edge from every
    monotone state of up to two placed objects, and a beam-2 search
    without colour, against the oracle."""
    meshes, scene, gt, cands = _random_world(seed)
    rng = np.random.default_rng(950 + seed)
    flags = int(rng.choice([oracle.MARK_OCCLUDERS, 0])) | int(rng.choice([0, oracle.USE_RGB])) | \
        int(rng.choice([oracle.VOL_AABB, oracle.VOL_CYL, oracle.VOL_LABEL]))
    stride, delta = int(rng.choice([1, 2, 3])), float(rng.choice([4.0, 7.5, 12.0]))
    rgb = bool(flags & oracle.USE_RGB)
    say(f"msg random world {seed}: flags {flags}, stride {stride}, delta {delta}")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, scene.labels, delta_mm=delta, tau_c=15.0, flags=flags,
                        stride=stride)
    mids = [ctx.load_mesh(m.xyz, m.tri, m.rgb) for m in meshes]
    tc = [_cuda(c) for c in cands]
    kw = dict(delta_mm=delta, tau_c=15.0, flags=flags, stride=stride)
    states = [()]
    for o in range(3):
        v = oracle.msg_expand(scene, [], meshes[o], cands[o], label=o + 1, **kw)[0]
        states += [((o, int(k)),) for k in np.flatnonzero(v)[:2]]
    for (o1, k1) in [st[0] for st in states[1:4]]:
        for o in range(3):
            if o == o1:
                continue
            v = oracle.msg_expand(scene, [(meshes[o1], o1 + 1, cands[o1][k1])], meshes[o], cands[o], label=o + 1,
                                  **kw)[0]
            states += [((o1, k1), (o, int(k))) for k in np.flatnonzero(v)[:1]]
    checked = 0
    for seq in states:
        placed = {o for o, _ in seq}
        gstate = [(mids[o], o + 1, cands[o][k]) for o, k in seq]
        ostate = [(meshes[o], o + 1, cands[o][k]) for o, k in seq]
        for o in range(3):
            if o in placed:
                continue
            got = ctx.msg_expand(sid, gstate, mids[o], tc[o], label=o + 1)
            exp = oracle.msg_expand(scene, ostate, meshes[o], cands[o], label=o + 1, threads=THREADS, **kw)
            check_edges(got, exp, rgb, f"world {seed} state {seq} object {o}")
            checked += 1
    ctx.drop_scene(sid)
    sid = ctx.set_scene(scene.K, scene.depth, None, scene.labels, delta_mm=delta, flags=flags & ~oracle.USE_RGB,
                        stride=stride)
    got = ctx.msg_search(sid, [(mids[o], o + 1, tc[o]) for o in range(3)], beam=2)
    exp = oracle.msg_search(scene, [(meshes[o], o + 1, cands[o]) for o in range(3)], beam=2, delta_mm=delta,
                            flags=flags & ~oracle.USE_RGB, stride=stride, threads=THREADS)
    ctx.drop_scene(sid)
    for m in mids:
        ctx.unload_mesh(m)
    assert got == exp, (got, exp)
    assert checked >= 6


def test_search_recovers_the_generating_scene(ctx):
    meshes, scene, gt, cands = _world(seed=2)
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, scene.labels, delta_mm=DELTA, tau_c=20.0,
                        flags=oracle.MARK_OCCLUDERS | oracle.USE_RGB)
    mids = [ctx.load_mesh(m.xyz, m.tri, m.rgb) for m in meshes]
    (cost, seq), scored = ctx.msg_search(sid, [(mids[o], o + 1, _cuda(cands[o])) for o in range(3)], beam=0)
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    assert sorted(seq) == [(0, 0), (1, 0), (2, 0)]
    assert [o for o, _ in seq].index(0) < [o for o, _ in seq].index(1)
    assert scored > 12


def test_refuses_bad_states_and_flags(ctx):
    meshes, scene, gt, cands = _world()
    sid = ctx.set_scene(scene.K, scene.depth, None, scene.labels, delta_mm=DELTA, flags=oracle.MARK_OCCLUDERS)
    mids = [ctx.load_mesh(m.xyz, m.tri, None) for m in meshes]
    t1 = _cuda(cands[2])
    # object 0 stands in front of object 1: placing 1 first, then 0, is not monotone
    with pytest.raises(pk.PerchError, match="monotone"):
        ctx.msg_expand(sid, [(mids[1], 2, gt[1]), (mids[0], 1, gt[0])], mids[2], t1, label=3)
    sid2 = ctx.set_scene(scene.K, scene.depth, None, scene.labels, delta_mm=DELTA, jo="nn")
    with pytest.raises(pk.PerchError, match="JO_NN"):
        ctx.msg_expand(sid2, [], mids[2], t1, label=3)
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    ctx.drop_scene(sid2)


@pytest.mark.parametrize("volume", ["aabb", "label"])
def test_cfg2_sampled_edges(ctx, volume):
    """640x480 cfg2 scene: two objects placed at their generating poses, the
    third object's 6,400 candidates scored on the GPU; a seeded sample of
    them (and the generating pose) against the oracle."""
    w = make_config(2, 0)
    s = w.scene
    flags = oracle.USE_RGB | (oracle.MARK_OCCLUDERS if w.mark_occluders else 0) | \
        (oracle.VOL_LABEL if volume == "label" else 0)
    say(f"msg cfg2 sampled edges: {volume}")
    sid = ctx.set_scene(s.K, s.depth, s.rgb, s.labels, delta_mm=w.delta_mm, tau_c=w.tau_c, flags=flags)
    mids = {k: ctx.load_mesh(m.xyz, m.tri, m.rgb) for k, m in enumerate(w.meshes)}
    objs = w.objects
    placed = [(objs[0].mesh, objs[0].label, objs[0].gt_pose), (objs[1].mesh, objs[1].label, objs[1].gt_pose)]
    o = objs[2]
    got = ctx.msg_expand(sid, [(mids[m], lab, p) for m, lab, p in placed], mids[o.mesh], _cuda(o.poses), label=o.label)
    got = [t.cpu().numpy() for t in got]
    rng = np.random.default_rng(9)
    sel = np.sort(rng.choice(o.poses.shape[0], 14, replace=False))
    poses = np.concatenate([o.poses[sel], o.gt_pose.reshape(1, 12).astype(np.float32)])
    exp = oracle.msg_expand(s, [(w.meshes[m], lab, p) for m, lab, p in placed], w.meshes[o.mesh], poses,
                            label=o.label, delta_mm=w.delta_mm, tau_c=w.tau_c, flags=flags, threads=THREADS)
    g_gt = ctx.msg_expand(sid, [(mids[m], lab, p) for m, lab, p in placed], mids[o.mesh],
                          _cuda(o.gt_pose.reshape(1, 12)), label=o.label)
    g_gt = [t.cpu().numpy() for t in g_gt]
    for m in mids.values():
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    sub = [np.concatenate([a[sel], b]) for a, b in zip(got, g_gt)]
    check_edges([torch.from_numpy(a) for a in sub], exp, True, f"cfg2 {volume}")
    assert exp[0].sum() > 0 and exp[3].max() > 100


def test_cfg2_search_matches_oracle(ctx):
    """A width-2 search at full resolution: the 640x480 cfg2 scene, its first
    three objects with six seeded candidates each, depth only with label
    volumes (exact costs): the oracle's goal and successor count."""
    w = make_config(2, 0)
    s = w.scene
    flags = oracle.MARK_OCCLUDERS | oracle.VOL_LABEL
    rng = np.random.default_rng(21)
    objs = w.objects[:3]
    cands = [np.ascontiguousarray(o.poses[np.sort(rng.choice(o.poses.shape[0], 6, replace=False))]) for o in objs]
    say("msg cfg2 search, beam 2")
    sid = ctx.set_scene(s.K, s.depth, None, s.labels, delta_mm=w.delta_mm, flags=flags)
    mids = [ctx.load_mesh(w.meshes[o.mesh].xyz, w.meshes[o.mesh].tri, None) for o in objs]
    got = ctx.msg_search(sid, [(m, o.label, _cuda(c)) for m, o, c in zip(mids, objs, cands)], beam=2)
    for m in mids:
        ctx.unload_mesh(m)
    ctx.drop_scene(sid)
    say(f"  GPU: {got}; oracle search")
    exp = oracle.msg_search(s, [(w.meshes[o.mesh], o.label, c) for o, c in zip(objs, cands)], beam=2,
                            delta_mm=w.delta_mm, flags=flags, threads=THREADS)
    assert got == exp, (got, exp)
    assert got[0] is not None


def test_device_tile_successors_match_oracle(ctx):
    """Successors whose raster tile exceeds the LDS (an object 170-200 mm from
    the camera over a 320x240 image) take the device-memory tile: as root
    edges, as the placed state with the far object behind it, and as
    successors that would occlude the far object (not monotone)."""
    from test_oracle_icp import K_HI, _scene_and_gt
    m, scene, gt = _scene_and_gt(0, K_HI)
    near = []
    for tz in (170.0, 200.0):
        P = gt.reshape(12).astype(np.float32).copy()
        P[11] = tz
        near.append(P)
    near = np.stack(near)
    far = gt.reshape(1, 12).astype(np.float32)
    flags = oracle.MARK_OCCLUDERS | oracle.USE_RGB
    say("msg device-tile successors")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, delta_mm=5.0, tau_c=20.0, flags=flags)
    mid = ctx.load_mesh(m.xyz, m.tri, m.rgb)
    kw = dict(delta_mm=5.0, tau_c=20.0, flags=flags, threads=THREADS)
    cases = [([], near, "root edges"), ([(near[0], 1)], far, "far object behind a near state"),
             ([(far[0], 1)], near, "near successors of the far state")]
    for state, cands, what in cases:
        got = ctx.msg_expand(sid, [(mid, lab, p) for p, lab in state], mid, _cuda(cands), label=2)
        exp = oracle.msg_expand(scene, [(m, lab, p) for p, lab in state], m, cands, label=2, **kw)
        check_edges(got, exp, True, what)
        if what == "root edges":
            assert exp[0].all() and exp[3].min() > 20000           # |dR \ C|: tiles beyond the LDS
        elif what == "far object behind a near state":
            assert exp[0].all() and exp[2][0] > 0
        else:
            assert not exp[0].any()
    ctx.unload_mesh(mid)
    ctx.drop_scene(sid)


def _row_of_boxes(K, z, n):
    """Boxes side by side from the nearest to the farthest, each a little
    behind the one before, the first and the last partly outside the image."""
    from tiny_meshes import box, pose_matrix, rot_x
    mesh = box((-35, -45, -30), (35, 45, 30), n=2, rgb_seed=4)
    half = 0.5 * K[0] / K[2]
    zs = [z + 120.0 * k for k in range(n)]                # farther than a box is deep: each state is monotone
    return mesh, [pose_matrix(rot_x(0.3), (half * zs[k] * (2 * k / (n - 1) - 1), 10.0 * (k % 3) - 10.0, zs[k]))
                  for k in range(n)]


@pytest.mark.parametrize("rgb", [False, True])
@pytest.mark.parametrize("n", [2, 7, 12])
def test_states_of_many_objects(ctx, n, rgb):
    """The nearest points of a state are brought up to date once for all its
    objects: the scores of a successor beside them, for states that cover a
    part of the image and all of it, one of whose objects adds no point."""
    from tiny_meshes import TScene
    K = (150, 110, 160.0, 155.0, 75.0, 55.0)
    mesh, poses = _row_of_boxes(K, 420.0, n)
    rng = np.random.default_rng(n)
    depth = np.zeros((110, 150), np.int64)
    col = np.zeros((110, 150, 3), np.uint8)
    for P in poses[::-1]:
        d, _, c = oracle.render(mesh, P, K)
        depth, col = np.where(d > 0, d, depth), np.where((d > 0)[..., None], c, col)
    depth = np.where(depth > 0, depth + rng.integers(-4, 5, depth.shape), 0).astype(np.uint16)
    gone = poses[0].copy()
    gone[3] += 4000.0                                     # beside the image: draws nothing
    placed = poses[:-1][: n // 2] + [gone] + poses[:-1][n // 2:]
    cand = np.stack([poses[-1]] * 12).astype(np.float32)
    cand[:, [3, 7, 11]] += rng.normal(0, 6, (12, 3)).astype(np.float32)
    flags = oracle.MARK_OCCLUDERS | (oracle.USE_RGB if rgb else 0)
    say(f"state of {len(placed)} objects, rgb {rgb}")
    sid = ctx.set_scene(K, depth, col, delta_mm=12.0, tau_c=20.0, flags=flags)
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    got = ctx.msg_expand(sid, [(mid, 1, P) for P in placed], mid, _cuda(cand), label=2)
    torch.cuda.synchronize()
    exp = oracle.msg_expand(TScene(K, depth, col), [(mesh, 1, P) for P in placed], mesh, cand, label=2, delta_mm=12.0,
                            tau_c=20.0, flags=flags, threads=THREADS)
    check_edges(got, exp, rgb, f"{n} boxes")
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)
    assert exp[0].any() and exp[4].max() > 0


def test_time_of_a_state_does_not_grow_with_its_objects_area(ctx):
    """A state of 24 objects, each as large as the image, at delta 30 mm takes
    little more than one of a single such object: what an object adds is its
    raster and composition (some 20 us), not a pass over all neighbour windows
    (2 ms).  With such a pass for each object the two were 6.5 apart."""
    from tiny_meshes import box, pose_matrix, rot_x
    K = (640, 480, 525.0, 525.0, 320.0, 240.0)
    h, z = 240, 700
    cube = box((-h, -h, -h), (h, h, h), n=10, rgb_seed=8)
    d, _, c = oracle.render(cube, pose_matrix(rot_x(0.5), (10, -5, z)), K)
    d = np.where(d > 0, d, z + h + 100).astype(np.uint16)
    sid = ctx.set_scene(K, d, c, delta_mm=30.0, tau_c=20.0)
    mid = ctx.load_mesh(cube.xyz, cube.tri, cube.rgb)
    ms = []
    for n in (1, 24):
        state = [(mid, 0, pose_matrix(rot_x(0.5), (10 + 3 * k, -5, z + 5 * h * k))) for k in range(n)]
        t = _cuda(np.stack([pose_matrix(rot_x(0.5), (10 + k, -5, z + 5 * h * n)) for k in range(8)]))
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ctx.msg_expand(sid, state, mid, t, label=0)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        ms.append(sorted(times)[3])
    say(f"state of 1 object {ms[0]:.2f} ms, of 24 {ms[1]:.2f} ms")
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)
    assert ms[1] < 2.5 * ms[0]
