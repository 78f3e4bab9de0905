"""Timing cases of the pose-scoring library, through its public Python entry points.

Each case is what a program of this library does over and over: score, search,
batch, prepare a new scene, refine candidates, or search the scene tree.  The
scenes follow the package's own workloads (table-top objects of its five
procedural shapes, a camera 0.8 m away, 2 mm depth noise, 5/255 colour noise),
with sizes of its configurations: 320x240 depth-only grids, 640x480 RGB grids
of 6,400 candidates an object, 6-DoF perturbations of 20k-triangle meshes, and
uneven many-scene batches.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) resident meshes, scene, candidates (on the GPU)
    run(state)          one pass
    work(case)          bytes and operations a pass cannot do without
    exact(case, seed)   the counts by plain numpy (depth-only scoring)
"""
import math

import numpy as np
import torch

import paper_2008_00326_amd as pk
from paper_2008_00326_amd.workloads import meshes as M
from paper_2008_00326_amd.workloads import scenes as S
from paper_2008_00326_amd.workloads import sensor

BASE = dict(width=640, height=480, objects=1, tris=2000, poses=64, dof=3, spread=285.0, rgb=True, delta=10.0, tau=20.0,
            volume="aabb", jo="exact", stride=1)
REFINE = dict(volume="label", rho=20.0, iterations=10, icp_stride=2)


def _case(name, kind, **kw):
    return {"name": name, "kind": kind, **BASE, **kw}


def listed():
    return [
        # one hypothesis checked, as a tracker or a grasp planner does: the smallest call, latency alone
        _case("verify_one_pose", "score", poses=1, spread=20.0),
        # the depth-only table-top search: one 1.2k-triangle object, 320x240, 512 candidates
        _case("grid_depth_512", "score", width=320, height=240, tris=1232, poses=512, spread=70.0, rgb=False, tau=0.0),
        # an odd-sized image and mesh with the thresholds that the paper quotes, 6-DoF, every second pixel rendered
        _case("odd_333_stride2", "score", width=427, height=321, tris=5003, poses=333, dof=6, delta=7.5, tau=12.5,
              stride=2),
        # a few proposals for each object, the minimum wanted on the host: short searches, launch latency and
        # a device that a pose per work-group cannot fill
        _case("search_5x32", "search", objects=5, tris=4000, poses=32),
        # the full RGB search: 5 objects of 6,400 candidates in one launch; the largest case
        _case("grid_rgb_32k", "joint", objects=5, tris=4000, poses=6400),
        # 6-DoF refinement sampling with dense meshes
        _case("perturb_6dof_8k", "joint", objects=4, tris=20000, poses=2048, dof=6),
        # nearest-neighbour marking with the inscribed cylinder: the paper's own J_o kernel and volume
        _case("nn_cylinder_6k", "joint", objects=5, tris=4000, poses=1200, volume="cyl", jo="nn"),
        # uneven scenes in one captured graph launch: 1 to 6 objects, 200 to 3,000 candidates, 500 to 50k triangles
        _case("graph_uneven_6", "graph", scenes=6, objects=6, tris=50000, poses=3000),
        # a request with a new image: scene preparation, a short labelled search, release
        _case("new_scene_64", "scene", objects=4, tris=4000, poses=64, volume="label"),
        # point-to-point ICP of table-top candidates against the object's segment
        _case("icp_3dof_1600", "refine", tris=4000, poses=1600, spread=60.0, method="point", **REFINE),
        # plane-to-plane GICP of the best 6-DoF proposals of one object
        _case("gicp_6dof_128", "refine", tris=20000, poses=128, dof=6, method="plane", **REFINE),
        # the sequential tree search over three objects
        _case("tree_3x400_beam4", "tree", objects=3, tris=3000, poses=400, beam=4, volume="label"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["score", "search", "joint", "graph", "scene", "refine", "tree"])
    w = _log_int(rng, 160, 640)
    c = {"kind": kind, **BASE, "width": w, "height": max(120, int(w * rng.uniform(0.6, 0.8))),
         "tris": _log_int(rng, 300, 20000), "dof": rng.choice([3, 6]), "spread": round(rng.uniform(40.0, 285.0), 1),
         "rgb": rng.random() < 0.7, "delta": round(rng.uniform(5.0, 12.0), 2), "tau": round(rng.uniform(10.0, 25.0), 2),
         "volume": rng.choice(["aabb", "aabb", "cyl", "label"]), "jo": rng.choice(["exact", "exact", "nn"]),
         "stride": rng.choice([1, 1, 2, 3])}
    if kind == "score":
        c.update(poses=_log_int(rng, 1, 3000))
    elif kind == "search":
        c.update(objects=rng.randint(1, 8), poses=_log_int(rng, 4, 400))
    elif kind == "joint":
        k = rng.randint(1, 8)
        c.update(objects=k, poses=_log_int(rng, 100, 12000 // k))
    elif kind == "graph":
        c.update(scenes=rng.randint(2, 5), objects=rng.randint(1, 5), poses=_log_int(rng, 32, 2000))
    elif kind == "scene":
        c.update(objects=rng.randint(1, 5), poses=_log_int(rng, 16, 256))
    elif kind == "refine":
        m = rng.choice(["point", "plane"])
        c.update(REFINE, method=m, dof=6 if m == "plane" else c["dof"], jo="exact", spread=round(rng.uniform(20, 80), 1),
                 poses=_log_int(rng, 16, 1000 if m == "point" else 256), rho=round(rng.uniform(8.0, 25.0), 1),
                 iterations=rng.randint(3, 15), icp_stride=rng.randint(1, 3))
    else:
        c.update(objects=rng.randint(2, 3), poses=_log_int(rng, 30, 300), jo="exact", beam=rng.randint(1, 4))
    return c


# ---------------------------------------------------------------- inputs

def _poses(rng, rig, case, n, R_wo, t_wo, three):
    """n candidates, n x 12 float32: uniform over the table patch with any yaw
    (3-DoF), or perturbations (15 mm, 10 degrees) of the object's own pose and
    of three random rotations (6-DoF)."""
    R_cw, c = rig
    if case["dof"] == 3:
        yaw = rng.uniform(0, 2 * np.pi, n)
        R = np.zeros((n, 3, 3))
        R[:, 0, 0] = R[:, 1, 1] = np.cos(yaw)
        R[:, 1, 0] = np.sin(yaw)
        R[:, 0, 1] = -R[:, 1, 0]
        R[:, 2, 2] = 1.0
        s = case["spread"]
        t = np.concatenate([rng.uniform(-s, s, (n, 2)), np.zeros((n, 1))], 1)
        if s < 100.0:      # a patch around the object itself
            t[:, :2] += t_wo[:2]
    else:
        w = rng.normal(0, np.radians(10.0), (n, 3))
        th = np.maximum(np.linalg.norm(w, axis=1), 1e-12)
        k = w / th[:, None]
        K = np.zeros((n, 3, 3))
        K[:, 2, 1], K[:, 0, 2], K[:, 1, 0] = k[:, 0], k[:, 1], k[:, 2]
        K -= K.transpose(0, 2, 1)
        E = np.eye(3) + np.sin(th)[:, None, None] * K + (1 - np.cos(th))[:, None, None] * (K @ K)
        seeds = np.stack([R_wo] + three)
        R = seeds[np.arange(n) % 4] @ E
        t = t_wo + rng.normal(0, 15.0, (n, 3))
    P = np.zeros((n, 3, 4))
    P[:, :, :3] = R_cw @ R
    P[:, :, 3] = (t - c) @ R_cw.T
    return P.reshape(n, 12).astype(np.float32)


def _table():
    t = M.box(1600.0, 1600.0, 20.0, 12)
    xyz = t.xyz.copy()
    xyz[:, 2] -= 20.0
    return M.Mesh(xyz, t.tri, np.full((t.n_verts, 3), 128, np.uint8), "table")


def _scene(rng, case, meshes, counts):
    """One observed image of the meshes on the table and, per mesh, its
    label and candidates."""
    W, H = case["width"], case["height"]
    f = 525.0 * W / 640.0
    K = (W, H, f, f, W / 2.0, H / 2.0)
    rig = S.camera_rig()
    table = _table()
    parts = [(table, S.table_pose(rig, 0, 0, 0), 0)]
    cells = rng.permutation(9)[:len(meshes)]
    objs = []
    for k, m in enumerate(meshes):
        xy = np.array([(cells[k] % 3 - 1) * 150.0, (cells[k] // 3 - 1) * 150.0]) + rng.uniform(-20, 20, 2)
        R = S.rot_z(rng.uniform(0, 2 * np.pi))
        if case["dof"] == 6:
            R = R @ [np.eye(3), S.rot_x(np.pi / 2), S.rot_y(np.pi / 2)][int(rng.integers(0, 3))]
        t = np.array([xy[0], xy[1], -float((m.xyz.astype(np.float64) @ R.T)[:, 2].min())])
        parts.append((m, S.world_to_cam(rig, R, t), k + 1))
        objs.append((k + 1, _poses(rng, rig, case, counts[k], R, t, [S.random_rotation(rng) for _ in range(3)])))
    z, c, lab = sensor.cast(K, parts)
    valid = z > 0
    d = np.where(valid, np.clip(np.rint(z + rng.normal(0, 2.0, z.shape)), 1, 65534), 0).astype(np.uint16)
    rgb = np.clip(np.rint(c + rng.normal(0, 5.0, c.shape)), 0, 255).astype(np.uint8)
    return K, d, np.where(valid[..., None], rgb, 0).astype(np.uint8), lab, objs


def _inputs(case, seed):
    """Host inputs: the meshes, and per scene (K, depth, rgb, labels, [(mesh
    index, label, candidates)])."""
    rng = np.random.default_rng([int(seed), 20080326])
    uneven = case["kind"] == "graph"
    if uneven:
        lo = min(500, case["tris"])
        lib = [M.make_shape(M.SHAPES[k % 5], int(np.exp(rng.uniform(np.log(lo), np.log(case["tris"] + 1)))), rng)
               .with_colours(rng) for k in range(6)]
        out = []
        shape = np.random.default_rng([case["scenes"], case["objects"], case["poses"]])   # the batch's make-up
        for _ in range(case["scenes"]):
            ids = [int(x) for x in shape.integers(0, len(lib), shape.integers(1, case["objects"] + 1))]
            counts = [int(np.exp(shape.uniform(np.log(min(200, case["poses"])), np.log(case["poses"] + 1)))) for _ in ids]
            K, d, c, lab, objs = _scene(rng, case, [lib[i] for i in ids], counts)
            out.append((K, d, c, lab, [(i, o[0], o[1]) for i, o in zip(ids, objs)]))
        return lib, out
    kinds = rng.permutation(5)
    lib = [M.make_shape(M.SHAPES[kinds[k % 5]], case["tris"], rng).with_colours(rng) for k in range(case["objects"])]
    K, d, c, lab, objs = _scene(rng, case, lib, [case["poses"]] * len(lib))
    return lib, [(K, d, c, lab, [(i, o[0], o[1]) for i, o in enumerate(objs)])]


def _set(ctx, case, sc):
    K, d, c, lab, _ = sc
    return ctx.set_scene(K, d, c if case["rgb"] else None, lab if case["volume"] == "label" else None,
                         delta_mm=case["delta"], tau_c=case["tau"], use_rgb=case["rgb"], volume=case["volume"],
                         jo=case["jo"], stride=case["stride"])


def prepare(case, seed):
    lib, scenes = _inputs(case, seed)
    ctx = pk.Context()
    mids = [ctx.load_mesh(m.xyz, m.tri, m.rgb if case["rgb"] else None) for m in lib]
    st = {"case": case, "ctx": ctx, "host": scenes[0]}
    new = case["kind"] == "scene"
    items = []
    total = sum(len(poses) for sc in scenes for _, _, poses in sc[4])
    st["out"] = out = torch.empty((4, total), dtype=torch.int32, device="cuda")   # J_r, J_o, L, Q of every candidate
    at = 0
    for sc in scenes:
        sid = None if new else _set(ctx, case, sc)
        for i, label, poses in sc[4]:
            n = len(poses)
            items.append({"scene": sid, "mesh": mids[i], "label": label, "poses": torch.from_numpy(poses).cuda(),
                          **{k: out[q, at:at + n] for q, k in enumerate(("jr", "jo", "nr", "nq"))}})
            at += n
    st["items"] = items
    if case["kind"] == "graph":
        st["batch"] = ctx.batch(len(items), sum(it["poses"].shape[0] for it in items), case["width"] * case["height"])
        st["batch"].set(items)
    return st


def run(st):
    case, ctx, items = st["case"], st["ctx"], st["items"]
    kind, it = case["kind"], items[0]
    if kind == "score":
        return ctx.score_poses(it["scene"], it["mesh"], it["poses"], label=it["label"])
    if kind == "joint":
        ctx.score_batch(items)
        return st["out"]
    if kind == "search":
        return ctx.best_poses(it["scene"], [x["mesh"] for x in items], [x["label"] for x in items],
                              [x["poses"] for x in items])
    if kind == "graph":
        st["batch"].launch()
        return [*st["batch"].wait(), st["out"]]
    if kind == "scene":
        sid = _set(ctx, case, st["host"])
        ctx.score_batch([dict(x, scene=sid) for x in items])
        ctx.drop_scene(sid)
        return st["out"]
    if kind == "refine":
        return ctx.refine_poses(it["scene"], it["mesh"], it["poses"], label=it["label"], rho_mm=case["rho"],
                                iterations=case["iterations"], stride=case["icp_stride"], dof=case["dof"],
                                method=case["method"])
    goal, scored = ctx.msg_search(it["scene"], [(x["mesh"], x["label"], x["poses"]) for x in items], beam=case["beam"])
    cost, seq = goal if goal is not None else (-1, ())
    return [int(cost), int(scored), np.array(seq, np.int64).reshape(-1)]


# ---------------------------------------------------------------- work

def work(case):
    """Bytes: image, meshes and candidates read once, results written once.
    Operations, per candidate: 60 a triangle (set-up), 10 a pixel of its box,
    and for a rendered point its neighbour test and colour difference, for an
    observed point of the volume the same."""
    px = case["width"] * case["height"]
    f = 525.0 * case["width"] / 640.0
    side = 110.0 * f / 800.0                      # pixels across an object of 11 cm at 0.8 m
    box, seen = side * side, 0.6 * side * side / case["stride"] ** 2
    tests = 300 if case["rgb"] else 30
    kind, k, n, tris = case["kind"], case["objects"], case["poses"], case["tris"]
    scenes = case.get("scenes", 1)
    if kind == "graph":                           # means of the uneven draws
        k, lo = (1 + k) / 2, min(200, n)
        n = (n - lo) / math.log(n / lo) if n > lo else n
        lt = min(500, tris)
        tris = (tris - lt) / math.log(tris / lt) if tris > lt else tris
    per = 60 * tris + 10 * box + tests * 2 * seen
    img = px * (2 + (3 if case["rgb"] else 0) + (4 if case["volume"] == "label" else 0))
    total = scenes * k * n
    byts = scenes * img + min(scenes * k, 6 if kind == "graph" else k) * tris * (12 + 8) + total * (48 + 16)
    if kind == "refine":
        pts = 0.6 * side * side / case["icp_stride"] ** 2
        per = 60 * tris + 10 * box + 0.5 * case["iterations"] * pts * (100 if case["method"] == "point" else 300)
    if kind == "tree":                            # levels of the beam: every unplaced object of each kept state
        total = n * sum((1 if lv == 0 else case["beam"]) * (k - lv) for lv in range(k))
    if kind == "scene":
        byts += img + px * 300                    # the images go to the device; its neighbour table is written
        return {"bytes": byts, "flops": total * per + px * 500}
    return {"bytes": byts, "flops": total * per}


# ---------------------------------------------------------------- plain numpy

def _exact_pose(K, depth, kx, ky, m, P, case):
    """(J_r, J_o, L, Q) of one pose by the definitions: a z-buffer of whole
    millimetres over 8 sub-pixel bits with the top-left rule, points in 1/16
    mm, exact radius tests over every pixel offset that can hold a neighbour."""
    W, H, fx, fy, cx, cy = K
    R, t = P.reshape(3, 4)[:, :3], P.reshape(3, 4)[:, 3]
    dq, delta, N = int(round(16 * case["delta"])), case["delta"], W * H
    v = m.xyz.astype(np.float64)
    X = [((R[a, 0] * v[:, 0] + R[a, 1] * v[:, 1]) + R[a, 2] * v[:, 2]) + t[a] for a in range(3)]
    iz = 1.0 / X[2]
    U = np.rint(256 * ((fx * X[0]) * iz + cx)).astype(np.int64)[m.tri]
    V = np.rint(256 * ((fy * X[1]) * iz + cy)).astype(np.int64)[m.tri]
    z = iz[m.tri]

    def edge(a, b, px, py):
        return (V[:, b] - V[:, a]) * (px - U[:, a]) - (U[:, b] - U[:, a]) * (py - V[:, a])

    area = edge(0, 1, U[:, 2], V[:, 2])
    sel = area > 0
    U, V, z, area = U[sel], V[sel], z[sel], area[sel]
    i0, j0 = np.maximum(-(-U.min(1) // 256), 0), np.maximum(-(-V.min(1) // 256), 0)
    i1, j1 = np.minimum(U.max(1) // 256, W - 1), np.minimum(V.max(1) // 256, H - 1)
    buf = np.full(N, 1 << 20, np.int64)
    for dj in range(int((j1 - j0).max(initial=-1)) + 1):
        for di in range(int((i1 - i0).max(initial=-1)) + 1):
            i, j = i0 + di, j0 + dj
            w = [edge(1, 2, 256 * i, 256 * j), edge(2, 0, 256 * i, 256 * j), edge(0, 1, 256 * i, 256 * j)]
            ok = (i <= i1) & (j <= j1)
            for e, (a, b) in enumerate(((1, 2), (2, 0), (0, 1))):
                dy, dx = V[:, b] - V[:, a], U[:, b] - U[:, a]
                ok &= w[e] >= np.where((dy > 0) | ((dy == 0) & (dx < 0)), 0, 1)
            if ok.any():
                s = (w[0] * z[:, 0] + w[1] * z[:, 1])[ok] + (w[2] * z[:, 2])[ok]
                d = np.rint(area[ok] / s).astype(np.int64)
                np.minimum.at(buf, (j * W + i)[ok][(d >= 1) & (d <= 65534)], d[(d >= 1) & (d <= 65534)])
    dep = depth.reshape(-1).astype(np.int64)
    keep = buf < (1 << 20)
    keep &= ~((dep > 0) & (16 * dep + dq < 16 * buf))
    gj, gi = np.divmod(np.arange(N), W)
    keep &= (gi % case["stride"] == 0) & (gj % case["stride"] == 0)
    e = delta + 0.25
    near = max(1.0, float(buf[keep].min(initial=1 << 20)) - e)
    slope = 1.0 + ((max(cx, W - cx) / fx) ** 2 + (max(cy, H - cy) / fy) ** 2)
    reach = int(max(fx, fy) * e * math.sqrt(slope) / near) + 1
    r = np.flatnonzero(keep)
    rx, ry, rz = (np.rint(kx[gi[r]] * buf[r]).astype(np.int64), np.rint(ky[gj[r]] * buf[r]).astype(np.int64), 16 * buf[r])
    ox, oy, oz = np.rint(kx[gi] * dep).astype(np.int64), np.rint(ky[gj] * dep).astype(np.int64), 16 * dep
    inl, expl = np.zeros(len(r), bool), np.zeros(N, bool)
    for dj in range(-reach, reach + 1):
        for di in range(-reach, reach + 1):
            i, j = gi[r] + di, gj[r] + dj
            u = np.where((i >= 0) & (i < W) & (j >= 0) & (j < H), j * W + i, r)
            hit = (dep[u] > 0) & ((u != r) | ((di == 0) & (dj == 0)))
            hit &= (ox[u] - rx) ** 2 + (oy[u] - ry) ** 2 + (oz[u] - rz) ** 2 <= dq * dq
            inl |= hit
            expl[u[hit]] = True
    q = np.stack([ox / 16.0 - t[0], oy / 16.0 - t[1], dep - t[2]], 1) @ R
    lo, hi = m.xyz.min(0).astype(np.float64), m.xyz.max(0).astype(np.float64)
    inv = (dep > 0) & ((q >= lo - delta) & (q <= hi + delta)).all(1)
    return int((~inl).sum()), int((inv & ~expl).sum()), len(r), int(inv.sum())


def exact(case, seed):
    """Depth-only box-volume scoring of at most 512 small poses; the colour
    decisions are binary32 by definition, and the refinements and the tree
    take minutes in numpy."""
    if case["kind"] != "score" or case["rgb"] or case["volume"] != "aabb" or case["jo"] != "exact":
        return None
    if case["poses"] * case["width"] * case["height"] > 512 * 320 * 240 or case["tris"] * case["poses"] > 700000:
        return None
    lib, ((K, d, _, _, objs),) = _inputs(case, seed)
    f32 = np.float32
    kx = ((np.arange(K[0]) - float(f32(K[4]))) * 16.0) / float(f32(K[2]))
    ky = ((np.arange(K[1]) - float(f32(K[5]))) * 16.0) / float(f32(K[3]))
    K64 = (K[0], K[1]) + tuple(float(f32(x)) for x in K[2:])
    c = dict(case, delta=float(f32(case["delta"])))
    got = [_exact_pose(K64, d, kx, ky, lib[0], p.astype(np.float64), c) for p in objs[0][2]]
    return [np.array(x, np.int32) for x in zip(*got)]
