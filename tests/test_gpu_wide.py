"""Launches of few poses (each pose spread over many work-groups) against the
footprint-class kernels (a work-group per pose), over every form that both
accept: the counts must be equal, colour decisions included, since both take
them in the same binary32 steps.  An explicit tuning selects the class
kernels; the forms' own parity with the oracle is tested elsewhere."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import paper_2008_00326_amd as pk  # noqa: E402
from random_cases import random_case  # noqa: E402
from tiny_meshes import box, pose_matrix, rot_x  # noqa: E402


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


def both(ctx, sid, mid, poses, label=0):
    t = torch.from_numpy(np.ascontiguousarray(poses, np.float32)).cuda()
    out = []
    for tuning in (None, {"order": 2}):
        ctx.set_tuning(tuning)
        out.append(torch.stack(ctx.score_poses(sid, mid, t, label=label)).cpu().numpy())
    ctx.set_tuning(None)
    return out


FORMS = [dict(), dict(use_rgb=False), dict(jo="nn"), dict(jo="nn", use_rgb=False), dict(volume="cyl"),
         dict(volume="label"), dict(search="hash"), dict(search="knn2"), dict(stride=3), dict(mark_occluders=False),
         dict(delta_mm=40.0, use_rgb=False), dict(volume="label", jo="nn", stride=2)]


@pytest.mark.parametrize("form", FORMS, ids=lambda f: "-".join(f"{k}={v}" for k, v in f.items()) or "default")
@pytest.mark.parametrize("n", [1, 7, 48])
def test_forms_agree(ctx, form, n):
    mesh, scene, poses, p = random_case(20 + n)
    say(f"wide form {form}, {n} poses, {scene.K[0]}x{scene.K[1]}")
    lab = (scene.depth > 0).astype(np.int32)
    lab[:, : scene.K[0] // 2] *= 2
    kw = {"delta_mm": p["delta"], "tau_c": p["tau"], "use_rgb": True, **form}
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, lab, **kw)
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    a, b = both(ctx, sid, mid, poses[:n], label=1)
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)
    assert np.array_equal(a, b), (a - b)
    assert a[2].sum() > 0


@pytest.mark.parametrize("n", [383, 384, 385])
def test_either_side_of_the_limit(ctx, n):
    """Pose counts around the path's limit, poses off the image and behind
    the camera among them; several items of one launch and their minima."""
    mesh, scene, poses, p = random_case(3)
    rng = np.random.default_rng(n)
    many = np.stack([poses[k % len(poses)] for k in range(n)])
    many[:, [3, 7, 11]] += rng.normal(0, 15, (n, 3)).astype(np.float32)
    many[5, 3] += 5000.0
    many[6, 11] = -400.0
    many[7, 11] = 60.0
    say(f"wide limit: {n} poses")
    sid = ctx.set_scene(scene.K, scene.depth, scene.rgb, delta_mm=p["delta"], tau_c=p["tau"], use_rgb=True)
    mid = ctx.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    a, b = both(ctx, sid, mid, many)
    assert np.array_equal(a, b)
    t = torch.from_numpy(many).cuda()
    parts = [t[:100].contiguous(), t[100:101].contiguous(), t[101:].contiguous()]
    bi, bc = ctx.best_poses(sid, [mid] * 3, [0] * 3, parts)
    j = a[0] + a[1]
    for k, (lo, hi) in enumerate(((0, 100), (100, 101), (101, n))):
        assert (int(bi[k]), int(bc[k])) == (int(np.argmin(j[lo:hi])), int(j[lo:hi].min()))
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)


def test_footprints_beyond_the_lds(ctx):
    """An object close to the camera: a tile that no LDS holds, bands that
    overflow the key and list capacities."""
    K = (640, 480, 500.0, 510.0, 320.0, 240.0)
    cube = box((-100, -100, -100), (100, 100, 100), n=6, rgb_seed=8)
    P0 = pose_matrix(rot_x(0.3), (10, -5, 330))
    d, _, c = oracle.render(cube, P0, K)
    say("wide: large footprints")
    sid = ctx.set_scene(K, d, c, delta_mm=10.0, tau_c=20.0, use_rgb=True)
    mid = ctx.load_mesh(cube.xyz, cube.tri, cube.rgb)
    poses = np.stack([P0, pose_matrix(rot_x(0.3), (13, -4, 332)), pose_matrix(np.eye(3), (0, 0, 260)),
                      pose_matrix(np.eye(3), (-20, 10, 700))])
    a, b = both(ctx, sid, mid, poses)
    ctx.drop_scene(sid)
    ctx.unload_mesh(mid)
    assert np.array_equal(a, b)
    assert a[2].max() > 40960 and a[0].min() < a[2].max() // 10


@pytest.mark.parametrize("h,z,delta", [(80, 520, 10.0), (39, 250, 15.5), (35, 250, 15.5), (80, 900, 10.0)])
def test_lists_of_many_inliers(ctx, h, z, delta):
    """Every rendered point an inlier: the class kernels' work lists fill and
    are worked off several times, and near the camera the observed window
    is longer than a list entry's range."""
    K = (640, 480, 500.0, 510.0, 320.0, 240.0)
    cube = box((-h, -h, -h), (h, h, h), n=6, rgb_seed=11)
    P0 = pose_matrix(rot_x(0.2), (5, -4, z))
    d, _, c = oracle.render(cube, P0, K)
    say(f"lists: cube of {2 * h} mm at {z} mm, delta {delta}")
    for use_rgb in (True, False):
        sid = ctx.set_scene(K, d, c, delta_mm=delta, tau_c=10.0, use_rgb=use_rgb)
        mid = ctx.load_mesh(cube.xyz, cube.tri, cube.rgb)
        poses = np.stack([P0, pose_matrix(rot_x(0.2), (8, -3, z + 4)), pose_matrix(rot_x(0.25), (2, -6, z - 1))])
        a, b = both(ctx, sid, mid, poses)
        classes = ctx.last_classes(len(poses))
        ctx.drop_scene(sid)
        ctx.unload_mesh(mid)
        assert np.array_equal(a, b)
        assert a[2].max() > 4096 and (classes <= 1).any()
