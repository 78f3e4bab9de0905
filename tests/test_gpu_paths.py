"""Which kernels score a launch: the profiler's slots tell the few-poses path
(each pose spread over many work-groups) from the footprint-class kernels, and
each is compared with the oracle where it is known to have run."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2008_00326_amd as pk  # noqa: E402
from paper_2008_00326_amd.workloads import make_config  # noqa: E402
from random_cases import random_case  # noqa: E402
from tiny_meshes import TScene, box, pose_matrix, rot_x  # noqa: E402

PATHS = [(None, True), ({"order": 2}, False), ({"small_block": 256, "key_bands": 1}, False)]   # (tuning, few-poses path)


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = pk.Context(0)
    yield c
    c.set_tuning(None)
    c.close()


def score(ctx, sid, mid, poses, tuning, label=0):
    """Outputs of one call under a tuning, and whether it took the few-poses
    path (the class kernels otherwise)."""
    ctx.set_tuning(tuning)
    t = torch.from_numpy(np.ascontiguousarray(poses, np.float32)).cuda()
    ctx.profile(True)
    out = ctx.score_poses(sid, mid, t, label=label)
    torch.cuda.synchronize()
    slots = ctx.profile_read()
    ctx.profile(False)
    ctx.set_tuning(None)
    wide, classes = slots["score_wide"][1], slots["score_lds_small"][1]
    assert wide + classes == 1
    return [x.cpu().numpy() for x in out], wide == 1


def test_a_saved_tuning_can_be_set_again(ctx):
    """tuning() spells the defaults out; set again they are the defaults, and
    any other setting, a field of its default's value among them, is a tuning."""
    mesh, scene, poses, p = random_case(4)
    say("saved tuning")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, delta_mm=p["delta"], tau_c=p["tau"])
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    ctx.set_tuning(None)
    saved = ctx.tuning()
    other = dict(saved, grid=[saved["grid"][0] - 1] + saved["grid"][1:])
    ref = None
    for tuning, few in ((None, True), (saved, True), ({"order": 2}, False), (other, False), (saved, True)):
        out, wide = score(ctx, sid, mid, poses[:8], tuning)
        assert wide == few, tuning
        ref = ref or out
        assert all(np.array_equal(a, b) for a, b in zip(out, ref))
    ctx.set_tuning(other)
    assert ctx.tuning() == other
    ctx.set_tuning(saved)
    assert ctx.tuning() == saved
    ctx.set_tuning(None)
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)


# (scene options, poses of the largest launch that takes the few-poses path)
LIMITS = [(dict(), 384), (dict(stride=2), 384), (dict(search="hash"), 384), (dict(search="knn2"), 384),
          (dict(search="hash", delta_mm=30.0), 80), (dict(search="knn2", delta_mm=30.0), 80),
          (dict(search="hash", delta_mm=30.0, use_rgb=False, mark_occluders=False), 80), (dict(jo="nn"), None),
          (dict(jo="nn", delta_mm=30.0), None), (dict(jo="nn", delta_mm=90.0, use_rgb=False), None),
          (dict(search="hash", jo="nn"), 128), (dict(search="hash", jo="nn", delta_mm=30.0), 0),
          (dict(search="knn2", jo="nn", delta_mm=30.0), 0)]


@pytest.mark.parametrize("form,limit", LIMITS, ids=lambda v: "-".join(f"{a}={b}" for a, b in v.items()) if isinstance(v, dict) else str(v))
def test_either_side_of_a_scene_s_limit(ctx, form, limit):
    """What a band repeats of its neighbours' rows lowers the limit of the
    few-poses path: the path on either side of it, the same results."""
    K = (160, 120, 300.0, 300.0, 80.0, 60.0)
    mesh = box((-30, -20, -25), (30, 20, 25), n=4, rgb_seed=3)
    gt = pose_matrix(rot_x(0.4), (8, -5, 520))
    depth, _, rgb = oracle.render(mesh, gt, K)
    depth = np.where(depth > 0, depth, 620).astype(np.uint16)
    kw = {"delta_mm": 3.0, "tau_c": 20.0, "use_rgb": True, **form}
    sid = ctx.set_scene(K, depth, rgb, **kw)
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    wty = ctx.scene_info(sid)["window_y"]
    if limit is None:
        limit = min(240, max(16, 6000 // wty))
    elif form.get("search"):
        assert (wty > 16) == ("delta_mm" in form)       # the rule's two sides
    say(f"limit {form}: {limit} poses, window {wty}")
    rng = np.random.default_rng(limit)
    many = np.stack([gt] * (limit + 1)).astype(np.float32)
    many[:, [3, 7, 11]] += rng.normal(0, 8, (limit + 1, 3)).astype(np.float32)
    ref, wide = score(ctx, sid, mid, many, {"order": 2})
    assert not wide
    for n in (limit, limit + 1):
        if n == 0:
            continue
        out, wide = score(ctx, sid, mid, many[:n], None)
        assert wide == (n <= limit)
        assert all(np.array_equal(a, b[:n]) for a, b in zip(out, ref))
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)


def oracle_flags(rgb, occl=True, volume="aabb", jo="exact"):
    return ((oracle.USE_RGB if rgb else 0) | (oracle.MARK_OCCLUDERS if occl else 0)
            | (oracle.VOL_CYL if volume == "cyl" else 0) | (oracle.JO_NN if jo == "nn" else 0))


def check(got, exp, rgb, jo, what):
    """L and Q equal, without the colour term J_r and J_o too; with it, whose
    decisions are binary32, within a thousandth of the points tested."""
    assert np.array_equal(got[2], exp[2]) and np.array_equal(got[3], exp[3]), what
    if not rgb:
        assert np.array_equal(got[0], exp[0]) and np.array_equal(got[1], exp[1]), what
        return
    tol_r = np.ceil(0.001 * exp[2])
    assert np.all(np.abs(got[0] - exp[0]) <= tol_r), what
    assert np.all(np.abs(got[1] - exp[1]) <= np.ceil(0.001 * exp[3]) + (tol_r if jo == "nn" else 0)), what


@pytest.mark.parametrize("form", [dict(), dict(volume="cyl"), dict(jo="nn"), dict(jo="nn", volume="cyl"),
                                  dict(search="hash"), dict(search="knn2"), dict(search="hash", jo="nn")],
                         ids=lambda f: "-".join(f.values()) or "default")
@pytest.mark.parametrize("seed", range(6))
def test_each_path_matches_the_oracle(ctx, seed, form):
    mesh, scene, poses, p = random_case(60 + seed)
    poses = poses[:24]
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, delta_mm=p["delta"], tau_c=p["tau"], use_rgb=p["rgb"],
                        mark_occluders=p["occl"], stride=p["stride"], **form)
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    jo = form.get("jo", "exact")
    exp = oracle.score(mesh, scene, poses, delta_mm=p["delta"], tau_c=p["tau"], stride=p["stride"], threads=16,
                       flags=oracle_flags(p["rgb"], p["occl"], form.get("volume", "aabb"), jo))
    wty = ctx.scene_info(sid)["window_y"]
    for tuning, few in PATHS:
        say(f"case {60 + seed} {form} {tuning} wty {wty}")
        got, wide = score(ctx, sid, mid, poses, tuning)
        assert wide == (few and not (jo == "nn" and "search" in form and wty > 16))
        check(got, exp, p["rgb"], jo, (seed, form, tuning))
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)
    assert exp[2].sum() > 0


@pytest.mark.parametrize("form", [dict(), dict(use_rgb=False), dict(jo="nn"), dict(search="hash", use_rgb=False)],
                         ids=lambda f: "-".join(str(v) for v in f.values()) or "default")
def test_tiles_beyond_the_lds_by_the_class_kernels(ctx, form):
    """Poses whose tile and keys no LDS holds, scored by the kernel of the
    device-memory class and by the few-poses path: the oracle's counts."""
    K = (320, 240, 262.5, 262.5, 160.0, 120.0)
    cube = box((-100, -100, -100), (100, 100, 100), n=6, rgb_seed=8)
    P0 = pose_matrix(np.eye(3), (10, -5, 420))
    d, _, c = oracle.render(cube, P0, K)
    kw = {"use_rgb": True, **form}
    sid = ctx.set_scene(K, d, c, delta_mm=10.0, tau_c=20.0, **kw)
    mid = ctx.load_mesh(cube.xyz, cube.tri, cube.rgb)
    poses = np.stack([P0, pose_matrix(np.eye(3), (14, -2, 415)), pose_matrix(np.eye(3), (0, 0, 330)),
                      pose_matrix(np.eye(3), (-20, 10, 700))])
    jo = form.get("jo", "exact")
    exp = oracle.score(cube, TScene(K, d, c, None), poses, delta_mm=10.0, tau_c=20.0, threads=16,
                       flags=oracle_flags(kw["use_rgb"], jo=jo))
    for tuning, few in PATHS[:2]:
        say(f"beyond the LDS {form} {tuning}")
        got, wide = score(ctx, sid, mid, poses, tuning)
        assert wide == few
        assert 3 in ctx.last_classes(len(poses)).tolist()
        check(got, exp, kw["use_rgb"], jo, (form, tuning))
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)


@pytest.mark.parametrize("jo", ["exact", "nn"])
def test_poses_of_each_class_by_the_class_kernels(ctx, jo):
    """640x480 RGB: poses of every footprint class that the full launch
    assigns, scored a few at a time by the class kernels and by the few-poses
    path, against the oracle and the full launch."""
    w = make_config(2, 0)
    s = w.scene
    sid = ctx.set_scene(s.K, s.depth, s.rgb, delta_mm=w.delta_mm, tau_c=w.tau_c, use_rgb=True, jo=jo)
    rng = np.random.default_rng(17)
    seen = set()
    for o in w.objects[:3]:
        m = w.meshes[o.mesh]
        mid = ctx.load_mesh(m.xyz, m.tri, m.rgb)
        full, wide = score(ctx, sid, mid, o.poses, {"key_bands": 1}, label=o.label)
        assert not wide
        cls = ctx.last_classes(len(o.poses))
        seen |= set(cls.tolist())
        sel = np.concatenate([rng.choice(np.flatnonzero(cls == k), 2) for k in np.unique(cls)])
        exp = oracle.score(m, TScene(s.K, s.depth, s.rgb, None), o.poses[sel], delta_mm=w.delta_mm, tau_c=w.tau_c,
                           flags=oracle_flags(True, w.mark_occluders, jo=jo), label=o.label, threads=16)
        for tuning, few in PATHS:
            say(f"each class, {jo}, object {o.label}, {tuning}")
            got, wide = score(ctx, sid, mid, o.poses[sel], tuning, label=o.label)
            assert wide == few
            check(got, exp, True, jo, (o.label, tuning))
            assert all(np.array_equal(a, b[sel]) for a, b in zip(got, full))
        ctx.unload_mesh(mid)
    ctx.drop_scene(sid)
    assert seen >= ({0, 1, 2} if jo == "exact" else {0, 1})
