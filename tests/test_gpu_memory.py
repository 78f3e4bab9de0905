"""Device memory of resident objects and of the per-stream scratch: what is
dropped counts against the context's budget no longer."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2008_00326_amd as pk  # noqa: E402
from tiny_meshes import box, pose_matrix  # noqa: E402


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("search", ["hash", "table"])
@pytest.mark.parametrize("labels", [False, True])
def test_dropped_scenes_give_their_memory_back(search, labels):
    """A budget of a few scenes holds any number of them one after another."""
    K = (320, 240, 300.0, 300.0, 160.0, 120.0)
    rng = np.random.default_rng(1)
    depth = rng.integers(800, 830, (240, 320)).astype(np.uint16)
    rgb = rng.integers(0, 256, (240, 320, 3)).astype(np.uint8)
    lab = rng.integers(0, 3, (240, 320)).astype(np.int32) if labels else None
    say(f"budget: scenes with search={search}, labels={labels}")
    with pk.Context(0) as ctx:
        size = ctx.scene_info(ctx.set_scene(K, depth, rgb, lab, delta_mm=5.0, search=search))["device_bytes"]
    with pk.Context(0, hbm_budget_bytes=3 * size + (8 << 20)) as ctx:
        for _ in range(40):
            sid = ctx.set_scene(K, depth, rgb, lab, delta_mm=5.0, search=search)
            assert ctx.scene_info(sid)["device_bytes"] == size
            ctx.drop_scene(sid)


def test_a_refused_allocation_is_reported_once():
    """Scratch that no device holds is refused; the calls after it, the
    library's and torch's on the same thread, do not report it again."""
    K = (64, 48, 60.0, 60.0, 32.0, 24.0)
    cube = box((-30, -30, -30), (30, 30, 30), n=2)
    d = np.full((48, 64), 500, np.uint16)
    say("refused allocation")
    with pk.Context(0) as ctx:
        sid = ctx.set_scene(K, d, delta_mm=5.0)
        mid = ctx.load_mesh(cube.xyz, cube.tri)
        t = torch.from_numpy(np.stack([pose_matrix(np.eye(3), (0, 0, 520))] * 5).astype(np.float32)).cuda()
        ref = torch.stack(ctx.score_poses(sid, mid, t)).cpu()
        with pytest.raises(pk.PerchError) as e:
            ctx.batch(1, 1, (1 << 31) - 1)               # some 6 TB of device-memory slots
        assert e.value.status == -2, e.value
        assert torch.equal(torch.stack(ctx.score_poses(sid, mid, t)).cpu(), ref)
        with pytest.raises(pk.PerchError):
            ctx.batch(1, 1, (1 << 31) - 1)
        assert float((t + 1.0).sum()) == pytest.approx(float(t.double().sum()) + t.numel(), rel=1e-5)
