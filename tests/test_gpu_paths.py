"""Which kernels score a launch: the profiler's slots tell the few-poses path
(each pose spread over many work-groups) from the footprint-class kernels."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2008_00326_amd as pk  # noqa: E402
from random_cases import random_case  # noqa: E402


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
