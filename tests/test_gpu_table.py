"""The neighbour table of a scene against the voxel hash, the same exact
nearest neighbours by another search: equal counts, in both J_o modes and
with colour, for windows inside and outside what the table's listed-offset
fill takes (reach in depth up to 32 mm), ranges of several passes, rows and
columns that no block divides, and readings missing or at the ends."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2008_00326_amd as pk  # noqa: E402
from tiny_meshes import box, pose_matrix, rot_x  # noqa: E402


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def depth_image(kind, W, H):
    rng = np.random.default_rng(W + H)
    y, x = np.mgrid[:H, :W]
    d = {"flat": np.full((H, W), 620),
         "slant": 560 + 2 * x + y,
         "noise": rng.integers(590, 650, (H, W)),
         "steps": np.where((x // 9 + y // 11) % 2, 615, 1300) + rng.integers(0, 3, (H, W)),
         "sparse": np.where(rng.random((H, W)) < 0.1, rng.integers(560, 700, (H, W)), 0)}[kind]
    return d.astype(np.uint16)


@pytest.mark.parametrize("size", [(1, 1), (63, 47), (130, 98)])
@pytest.mark.parametrize("delta", [0.4, 10.0, 32.0, 33.1])
@pytest.mark.parametrize("kind", ["flat", "slant", "noise", "steps", "sparse"])
def test_table_equals_hash(kind, delta, size):
    W, H = size
    f = 1.2 * max(W, 32)
    K = (W, H, f, 0.97 * f, 0.5 * W - 0.2, 0.5 * H + 0.3)
    d = depth_image(kind, W, H)
    rgb = np.random.default_rng(1).integers(0, 256, (H, W, 3)).astype(np.uint8)
    mesh = box((-150, -120, -40), (150, 120, 40), n=3, rgb_seed=3)
    poses = np.stack([pose_matrix(rot_x(0.1 * k), (4.0 * k, -3.0 * k, 600.0 + 25.0 * k)) for k in range(6)])
    t = torch.from_numpy(np.ascontiguousarray(poses, np.float32)).cuda()
    say(f"table {kind} delta {delta} {W}x{H}")
    c = pk.Context(0)
    mid = c.load_mesh(mesh.xyz, mesh.tri, mesh.rgb)
    for jo in ("exact", "nn"):
        out = []
        for search in ("table", "hash"):
            sid = c.set_scene(K, d, rgb, delta_mm=delta, tau_c=25.0, use_rgb=True, jo=jo, search=search)
            out.append(torch.stack(c.score_poses(sid, mid, t)).cpu().numpy())
            c.drop_scene(sid)
        assert np.array_equal(out[0], out[1]), (jo, out[0] - out[1])
    c.unload_mesh(mid)
    c.close()


@pytest.mark.parametrize("fy", [0.13, 40.0])
def test_pixels_far_from_square(fy):
    """A focal length in x of millions of pixels, in y of a fraction of one:
    the table is filled without a list of offsets as long as their ratio."""
    import oracle
    from tiny_meshes import TScene
    K = (4096, 4, 2.3e8, fy, 0.0, 2.0)
    rng = np.random.default_rng(5)
    d = rng.integers(64999, 65002, (4, 4096)).astype(np.uint16)
    d[:, 1000:] = 0
    mesh = box((0.05, -9e5, -0.5), (1.0, 9e5, 0.5), n=1)
    poses = np.stack([pose_matrix(np.eye(3), (0.01 * k, 0.0, 65000.0 + 0.5 * k)) for k in range(3)]).astype(np.float32)
    exp = oracle.score(mesh, TScene(K, d), poses, delta_mm=0.2, flags=oracle.MARK_OCCLUDERS, threads=8, search="window")
    assert exp[2].min() > 1000 and (0 < exp[0]).any() and (exp[0] < exp[2]).any()
    t = torch.from_numpy(poses).cuda()
    for search in ("table", "hash"):
        say(f"pixels of 1 : {2.3e8 / fy:.2g}, {search}")
        with pk.Context(0) as c:
            mid = c.load_mesh(mesh.xyz, mesh.tri)
            sid = c.set_scene(K, d, delta_mm=0.2, search=search)
            got = [x.cpu().numpy() for x in c.score_poses(sid, mid, t)]
        assert all(np.array_equal(a, b) for a, b in zip(got, exp)), (search, got, exp)
