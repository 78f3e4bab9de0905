"""Which kernels score a launch: the profiler's slots tell the few-poses path
(each pose spread over many work-groups) from the footprint-class kernels."""
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
