"""The work that a user of this library has it do, as measurable cases.

A case is a dict of plain values; `kind` names the public calls it goes
through:

  check    a batch of configurations against obstacles: flags, or flags and
           minimum signed distances (check_collisions)
  inflate  edges of the stored workloads inflated to certified sets in one
           call (inflate_edges)
  paths    piecewise-linear paths in sequence with the containment skip
           (inflate_paths)
  recover  a trajectory through loose sets: fine check of its points, the
           sets edited by the collisions found, its segments looked up
           (check_path, update_polytopes, segments_contained)
  map      a roadmap's nodes against every voxel, and the id lists
           (collision_map, collision_map_lists)
  predict  the learned self-collision screen on a batch (Surrogate.predict)
  grad     its training pass: loss and gradient of a batch
           (Surrogate.loss_grad)

Scenes are the stored workloads' (a subset of their obstacles keeps their
segments free, and so does a part of a segment), or drawn from the seed by the
same laws.  The number of samples N_p is given, never left to the tuner, so
that a case's sets do not depend on timing.
"""
import math

import numpy as np
import torch

import paper_2504_10783_amd as ezo
import workloads

DEV = "cuda:0"
ARMS = {"arm7": "sweep", "planar": "tiny", "boxes": "boxes", "point": "forest"}
# obstacle scenes of the checks: centres' box and radii (arm7, planar: the
# stored workloads' laws; boxes, point: the stored voxel spheres and discs)
SCENES = {"arm7": ((0.3, -0.5, 0.0), (1.3, 0.5, 1.0), 0.02, 0.08),
          "planar": ((-1.5, -1.5, 0.0), (1.5, 1.5, 0.0), 0.05, 0.15)}
# unadaptive tests a run of each workload takes (measured, typical)
ROUNDS = {"tiny": 2, "dof7": 4, "batched": 4, "boxes": 3, "forest": 2}
MAP_LO = (-1.5, -1.5, -0.5)
MAP_EXTENT = (3.04, 3.04, 2.0)
SEGMENT_STEP = 0.01
MOST_POINTS = 16384       # found collisions that a program takes
MOST_VOXELS = 600         # voxels per node that a program's table of ids has room for


def listed():
    return [
        # one planner query's worth of configurations (a few edges at a fine
        # step): the call's latency, its launches and the grid build
        dict(name="check 1000 flags", kind="check", arm="arm7", n=1000, n_obs=512, mode="flags", layout="rows",
             noalloc=True),
        # the raw checker's sweep: a large batch, flags only
        dict(name="check 4M flags", kind="check", arm="arm7", n=1 << 22, n_obs=1024, mode="flags", layout="rows",
             noalloc=False),
        # signed distances against the largest scene (clearances, labels)
        dict(name="check 256k distances", kind="check", arm="arm7", n=1 << 18, n_obs=4096, mode="sd", layout="rows",
             noalloc=False),
        # the box arm among voxel spheres and a table, an odd batch
        dict(name="check boxes", kind="check", arm="boxes", n=300001, n_obs=194, mode="sd", layout="coords",
             noalloc=False),
        # a small planar arm's edge: the shortest whole inflation
        dict(name="inflate planar edge", kind="inflate", scene="tiny", edges=1, n_obs=20, n_p=1000, iters=50),
        # one edge of the 7-DOF arm at the paper's N_p
        dict(name="inflate 7-DOF edge", kind="inflate", scene="dof7", edges=1, n_obs=512, n_p=10000, iters=50),
        # every edge of 8 paths in one call
        dict(name="inflate 96 edges", kind="inflate", scene="batched", edges=96, n_obs=2048, n_p=1000, iters=50),
        # the same paths in sequence, contained edges skipped
        dict(name="inflate 8 paths", kind="paths", scene="batched", paths=8, n_obs=2048, n_p=1000, iters=50),
        # lazy trajectory check and repair of 96 loose sets
        dict(name="recover 96 sets", kind="recover", scene="batched", edges=96, n_obs=2048, n_p=2000, per_edge=8),
        # the collision map of a 35 000-node roadmap over 8 cm voxels
        dict(name="map 35000 nodes", kind="map", arm="arm7", n=35000, side=0.08),
        # the screen on a million configurations, and one training pass
        dict(name="predict 1M", kind="predict", hidden=256, n=1 << 20),
        dict(name="gradient 4096", kind="grad", hidden=256, n=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("check", "check", "check", "inflate", "inflate", "inflate", "paths", "recover", "map",
                       "predict", "grad"))
    if kind == "check":
        arm = rng.choice(("arm7", "arm7", "arm7", "planar", "boxes", "point"))
        mode = rng.choice(("flags", "flags", "sd"))
        n_obs = {"arm7": _log_int(rng, 16, 4096), "planar": _log_int(rng, 4, 300), "boxes": rng.randint(20, 194),
                 "point": rng.randint(3, 15)}[arm]
        most = 1 << 22 if mode == "flags" else min(1 << 20, (1 << 30) // max(n_obs, 256))
        if arm == "boxes":
            most = 1 << 19
        return dict(kind=kind, arm=arm, n=_log_int(rng, 50, most), n_obs=n_obs, mode=mode,
                    layout=rng.choice(("rows", "rows", "coords")), noalloc=rng.random() < 0.3)
    if kind == "inflate":
        scene = rng.choice(("tiny", "dof7", "dof7", "batched", "batched", "boxes", "forest"))
        n_obs = {"tiny": rng.randint(4, 20), "dof7": _log_int(rng, 32, 512), "batched": _log_int(rng, 64, 2048),
                 "boxes": rng.randint(30, 194), "forest": rng.randint(5, 15)}[scene]
        edges = {"batched": _log_int(rng, 1, 96), "forest": rng.randint(1, 4)}.get(scene, 1)
        return dict(kind=kind, scene=scene, edges=edges, n_obs=n_obs, n_p=_log_int(rng, 500, 2000 if edges > 32 else 10000),
                    iters=rng.choice((50, 50, 3)))
    if kind == "paths":
        return dict(kind=kind, scene="batched", paths=rng.randint(1, 8), n_obs=_log_int(rng, 200, 2048),
                    n_p=_log_int(rng, 500, 1500), iters=50)
    if kind == "recover":
        return dict(kind=kind, scene="batched", edges=_log_int(rng, 4, 96), n_obs=_log_int(rng, 300, 2048), n_p=2000,
                    per_edge=rng.randint(3, 8))
    if kind == "map":
        return dict(kind=kind, arm=rng.choice(("arm7", "arm7", "boxes")), n=_log_int(rng, 500, 35000),
                    side=rng.choice((0.08, 0.08, 0.1, 0.16)))
    if kind == "predict":
        return dict(kind=kind, hidden=rng.choice((64, 128, 256)), n=_log_int(rng, 1000, 1 << 20))
    return dict(kind=kind, hidden=rng.choice((64, 128, 256)), n=64 * _log_int(rng, 1, 256))


def _cuda(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform_q(data, n, gen):
    lo, hi = _cuda(data["q_lo"]), _cuda(data["q_hi"])
    return lo + torch.rand((n, data["dof"]), generator=gen, device=DEV) * (hi - lo)


def _check_inputs(case, seed):
    """(stored data, configurations [n][dof], obstacles [n_obs][4])."""
    data = workloads.load(ARMS[case["arm"]])
    gen = _generator(seed)
    q = _uniform_q(data, case["n"], gen)
    if case["arm"] in SCENES:
        lo, hi, r0, r1 = SCENES[case["arm"]]
        lo, hi = torch.tensor(lo, device=DEV), torch.tensor(hi, device=DEV)
        u = torch.rand((case["n_obs"], 4), generator=gen, device=DEV)
        obs = torch.cat([lo + u[:, :3] * (hi - lo), r0 + u[:, 3:] * (r1 - r0)], dim=1)
    else:
        obs = _cuda(data["obstacles"])[torch.randperm(len(data["obstacles"]), generator=gen, device=DEV)[:case["n_obs"]]]
    return data, q, obs.contiguous()


def _scene(case, seed):
    """(stored data, obstacles, generator): a random subset of the scene's obstacles."""
    data = workloads.load(case["scene"])
    gen = _generator(seed)
    obs = _cuda(data["obstacles"])
    return data, obs[torch.randperm(len(obs), generator=gen, device=DEV)[:case["n_obs"]]].contiguous(), gen


def _part(edges, gen):
    """A random part of each segment (most of it), as a segment of its own."""
    t = torch.rand((len(edges), 2, 1), generator=gen, device=DEV) * 0.1
    v1, v2 = edges[:, :1], edges[:, 1:]
    return torch.cat([v1 + t[:, :1] * (v2 - v1), v2 - t[:, 1:] * (v2 - v1)], dim=1).contiguous()


def _params(case, data, seed, **more):
    p = dict(workloads.PARAMS[case["scene"]], n_p=case["n_p"], max_iters=case.get("iters", 50))
    p.update(more)
    return ezo.make_params(dof=data["dof"], seed=int(seed), **p)


def _result(E, cap, dof):
    """Output buffers a program keeps for its inflations, empty rows zero."""
    return ezo.InflateResult(torch.zeros((E, cap, dof), device=DEV), torch.zeros((E, cap), device=DEV),
                             torch.zeros(E, dtype=torch.int32, device=DEV),
                             torch.zeros(E, dtype=torch.int32, device=DEV), [])


def prepare(case, seed):
    ctx = ezo.Context(0)
    kind = case["kind"]
    if kind == "check":
        data, q, obs = _check_inputs(case, seed)
        if "env_boxes" in data:
            ctx.set_obstacle_boxes(data["env_boxes"])
        n = case["n"]
        s = dict(robot=ezo.Robot(ctx, workloads.robot(data)), obs=obs, q=q, how=dict(noalloc=case["noalloc"]),
                 flags=torch.zeros(n, dtype=torch.uint8, device=DEV), sd=None, sd_self=None)
        if case["layout"] == "coords":
            s["q"] = q.t().contiguous()
            s["how"].update(n=n, stride_n=1, stride_d=n)
        if case["mode"] == "sd":
            s["sd"], s["sd_self"] = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    elif kind == "inflate":
        data, obs, gen = _scene(case, seed)
        if "env_boxes" in data:
            ctx.set_obstacle_boxes(data["env_boxes"])
        e = _cuda(data["edges"])
        e = e[torch.randperm(len(e), generator=gen, device=DEV)[:case["edges"]].sort().values]
        prm = _params(case, data, seed)
        s = dict(robot=ezo.Robot(ctx, workloads.robot(data)), obs=obs, edges=_part(e, gen), params=prm,
                 out=_result(case["edges"], prm.face_capacity, data["dof"]))
    elif kind == "paths":
        data, obs, gen = _scene(case, seed)
        e, pid = data["edges"], data["path_id"]
        verts, counts = [], []
        for p in np.unique(pid)[:case["paths"]]:
            ep = _cuda(e[pid == p])
            # the path cut inside its first and its last segment
            t = torch.rand(2, generator=gen, device=DEV) * 0.3
            verts += [(ep[:1, 0] + t[0] * (ep[:1, 1] - ep[:1, 0])), ep[1:, 0],
                      (ep[-1:, 1] - t[1] * (ep[-1:, 1] - ep[-1:, 0]))]
            counts.append(len(ep) + 1)
        s = dict(robot=ezo.Robot(ctx, workloads.robot(data)), obs=obs, vertices=torch.cat(verts).contiguous(),
                 counts=counts, params=_params(case, data, seed))
    elif kind == "recover":
        data, obs, gen = _scene(case, seed)
        robot, dof, E, m = ezo.Robot(ctx, workloads.robot(data)), data["dof"], case["edges"], case["per_edge"]
        edges = _part(_cuda(data["edges"])[:E], gen)
        # sets after one iteration still hold collisions; rows are left for the repair
        prm = _params(case, data, seed, max_iters=1, face_capacity=2 * dof + 10 + 64)
        sets = ezo.inflate_edges(ctx, robot, obs, edges, prm, out=_result(E, prm.face_capacity, dof))
        pts = torch.zeros((E, dof, m), device=DEV)
        ezo.sample_polytopes(ctx, dof, sets.A, sets.b, sets.n_faces, edges, m, prm.n_mix, int(seed) + 7, 0, pts)
        way = torch.cat([edges[:, :1], pts.transpose(1, 2), edges[:, 1:]], dim=1).reshape(-1, dof).contiguous()
        s = dict(robot=robot, obs=obs, edges=edges, sets=sets, way=way,
                 segments=torch.stack([way[:-1], way[1:]], dim=1).contiguous(),
                 found=torch.zeros((MOST_POINTS, dof), device=DEV))
    elif kind == "map":
        data = workloads.load(ARMS[case["arm"]])
        side = case["side"]
        dims = [int(round(x / side)) for x in MAP_EXTENT]
        words = (case["n"] + 31) // 32
        s = dict(robot=ezo.Robot(ctx, workloads.robot(data)), q=_uniform_q(data, case["n"], _generator(seed)),
                 side=side, dims=dims, out=torch.zeros((int(np.prod(dims)), words), dtype=torch.int32, device=DEV),
                 ids=torch.zeros(case["n"] * MOST_VOXELS, dtype=torch.int32, device=DEV))
    else:
        data = workloads.load(ARMS["arm7"])
        q = _uniform_q(data, case["n"], _generator(seed))
        s = dict(screen=ezo.Surrogate(ctx, data["dof"], hidden=case["hidden"], seed=int(seed)), q=q)
        if kind == "predict":
            s["out"] = torch.zeros(case["n"], device=DEV)
        else:
            s["target"], s["tp"] = _screen_targets(q), ezo.make_train_params()
    s.update(kind=kind, ctx=ctx)
    return s


def _screen_targets(q):
    """Self distances of about the arm's spread: a smooth function of q in
    [-0.25, 0.45], about a third of them negative."""
    return (0.1 + 0.35 * torch.sin(1.3 * q[:, 1] + q[:, 3]) * torch.cos(q[:, 2] - 0.7 * q[:, 5])).contiguous()


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "check":
        ezo.check_collisions(ctx, s["robot"], s["obs"], s["q"], s["flags"], s["sd"], s["sd_self"], **s["how"])
        return s["flags"], s["sd"], s["sd_self"]
    if kind == "inflate":
        r = ezo.inflate_edges(ctx, s["robot"], s["obs"], s["edges"], s["params"], out=s["out"])
        return dict(A=r.A, b=r.b, n_faces=r.n_faces, status=r.status,
                    checks=r.stats.array["exact_checks"], iterations=r.stats.array["iterations"])
    if kind == "paths":
        r = ezo.inflate_paths(ctx, s["robot"], s["obs"], s["vertices"], s["counts"], s["params"])
        # rows past a set's faces are never written: they come back as zeros
        held = torch.arange(r.b.shape[1], device=DEV)[None, :] < r.n_faces[:, None]
        return dict(A=torch.where(held[..., None], r.A, 0.0), b=torch.where(held, r.b, 0.0), n_faces=r.n_faces,
                    status=r.status, covered_by=r.covered_by, checks=r.stats.array["exact_checks"])
    if kind == "recover":
        pts, found, total = ezo.check_path(ctx, s["robot"], s["obs"], s["way"], SEGMENT_STEP, point_capacity=MOST_POINTS)
        s["found"][:len(pts)] = pts                # the program's list of found collisions, of a fixed size
        old = s["sets"]
        sets = ezo.InflateResult(old.A.clone(), old.b.clone(), old.n_faces.clone(), old.status.clone(), [])
        added = ezo.update_polytopes(ctx, s["robot"], s["obs"], s["edges"], pts, sets)
        covered = ezo.segments_contained(ctx, sets.A, sets.b, sets.n_faces, s["segments"])
        return dict(points=s["found"], found=found, total=total, A=sets.A, b=sets.b, n_faces=sets.n_faces,
                    status=sets.status, added=added, covered=covered)
    if kind == "map":
        ezo.collision_map(ctx, s["robot"], s["q"], MAP_LO, s["side"], s["dims"], out=s["out"])
        offsets, ids = ezo.collision_map_lists(ctx, s["out"], s["q"].shape[0])
        s["ids"][:len(ids)] = ids                  # the program's table, of a fixed size
        return s["out"], offsets, s["ids"]
    if kind == "predict":
        s["screen"].predict(s["q"], s["out"])
        return s["out"]
    loss, grad = s["screen"].loss_grad(s["q"], s["target"], s["tp"])
    return dict(loss=loss, grad=grad)


def _check_flops(data, n_obs):
    """Forward kinematics of every sphere and box, and one pair test each."""
    dof, S, B = data["dof"], len(data["sphere_r"]), len(data.get("box_link", ()))
    return 60 * dof + 18 * S + 72 * B + (13 if n_obs else 0) * (S + B)


def work(case):
    kind = case["kind"]
    if kind == "check":
        data = workloads.load(ARMS[case["arm"]])
        n = case["n"]
        return dict(bytes=n * (4 * data["dof"] + 1 + (8 if case["mode"] == "sd" else 0)) + 16 * case["n_obs"],
                    flops=n * _check_flops(data, case["n_obs"]))
    if kind in ("inflate", "paths"):
        data = workloads.load(case["scene"])
        p, dof = workloads.PARAMS[case["scene"]], data["dof"]
        rounds = min(ROUNDS[case["scene"]], case["iters"])
        E = case["edges"] if kind == "inflate" else int(np.sum(np.isin(data["path_id"], np.unique(data["path_id"])[:case["paths"]])))
        rows = 2 * dof + p["n_f"] * (rounds - 1)
        # per round: the walks through the rows, the samples' checks, and a
        # tenth of them bisected
        per = case["n_p"] * (p["n_mix"] * rows * 4 * dof + (1 + 0.1 * (1 + p["n_b"])) * _check_flops(data, case["n_obs"]))
        return dict(bytes=16 * case["n_obs"] + E * (8 * dof + 4 * rows * (dof + 1) + 8), flops=E * rounds * per)
    if kind == "recover":
        data = workloads.load(case["scene"])
        dof, points = data["dof"], case["edges"] * (case["per_edge"] + 2) * 180
        return dict(bytes=16 * case["n_obs"] + 2 * case["edges"] * 4 * 24 * (dof + 1) + points * 4 * dof,
                    flops=1.5 * points * _check_flops(data, case["n_obs"]))
    if kind == "map":
        data = workloads.load(ARMS[case["arm"]])
        V = np.prod([int(round(x / case["side"])) for x in MAP_EXTENT])
        # the map written once and read once for the lists
        return dict(bytes=float(2 * V * ((case["n"] + 31) // 32) * 4), flops=case["n"] * _check_flops(data, 0))
    H, dof = case["hidden"], 7
    macs = case["n"] * (dof * H + 2 * H * H + H)
    if kind == "predict":
        return dict(bytes=case["n"] * 4 * (dof + 1) + 4 * H * H, flops=2 * macs)
    return dict(bytes=case["n"] * 4 * (dof + 1) + 2 * 4 * (2 * H * H + H * (dof + 4)), flops=6 * macs)


# ---- the same in 64 bits ----------------------------------------------------

def _frames(data, q):
    """Rotations [n][dof][3][3] and origins [n][dof][3] of every link."""
    n = q.shape[0]
    R = torch.eye(3, dtype=torch.float64, device=DEV).expand(n, 3, 3)
    p = torch.zeros((n, 3), dtype=torch.float64, device=DEV)
    kinds = data.get("joint_type", np.zeros(data["dof"], np.int32))
    Rs, ps = [], []
    for j in range(data["dof"]):
        a, d, al = (float(data[k][j]) for k in ("a", "d", "alpha"))
        th, d = (torch.zeros_like(q[:, j]), d + q[:, j]) if kinds[j] == 1 else (q[:, j], d + 0.0 * q[:, j])
        c, s, ca, sa, o = torch.cos(th), torch.sin(th), math.cos(al), math.sin(al), torch.zeros_like(th)
        M = torch.stack([c, -s * ca, s * sa, s, c * ca, -c * sa, o, o + sa, o + ca], dim=1).reshape(n, 3, 3)
        p = p + (R @ torch.stack([a * c, a * s, d], dim=1)[..., None])[..., 0]
        R = R @ M
        Rs.append(R)
        ps.append(p)
    return torch.stack(Rs, 1), torch.stack(ps, 1)


def _box_excess(R, c, h, x):
    """Signed distance of points x to boxes (R, c, h), broadcast."""
    d = x - c
    e = torch.stack([(R[..., 0, k] * d[..., 0] + R[..., 1, k] * d[..., 1] + R[..., 2, k] * d[..., 2]).abs() - h[..., k]
                     for k in range(3)], dim=-1)
    m = e.max(-1).values
    return torch.where(m <= 0, m, e.clamp(min=0).square().sum(-1).sqrt())


def _separation(Ra, ca, ha, Rb, cb, hb):
    """Separating-axis value of two boxes (3 + 3 face normals, 9 cross products)."""
    t = cb - ca
    best = torch.full(t.shape[:-1], -math.inf, dtype=torch.float64, device=DEV)
    axes = [(Ra[..., :, i], None) for i in range(3)] + [(Rb[..., :, i], None) for i in range(3)]
    axes += [(Ra[..., :, i], Rb[..., :, j]) for i in range(3) for j in range(3)]
    for u, v in axes:
        ok = None
        if v is not None:
            u = torch.linalg.cross(u.expand_as(t), v.expand_as(t))
            n2 = u.square().sum(-1)
            ok = n2 >= 1e-12
            u = u / n2.clamp(min=1e-300).sqrt()[..., None]
        u = u.expand_as(t)
        val = (t * u).sum(-1).abs()
        for R, h in ((Ra, ha), (Rb, hb)):
            val = val - sum(h[..., k] * (R[..., :, k] * u).sum(-1).abs() for k in range(3))
        best = torch.maximum(best, val if ok is None else torch.where(ok, val, -math.inf))
    return best


def _distances(data, q, obs):
    """Minimum signed distances (overall, self pairs) of q [n][dof]."""
    f = lambda k: _cuda(np.asarray(data[k], np.float64))
    n, inf = q.shape[0], math.inf
    R, p = _frames(data, q)
    env = torch.full((n,), inf, dtype=torch.float64, device=DEV)
    own = env.clone()
    link = torch.from_numpy(np.asarray(data["sphere_link"], np.int64)).to(DEV)
    if len(link):
        rad = f("sphere_r")
        cen = p[:, link] + (R[:, link] @ f("sphere_xyz")[..., None])[..., 0]
        for s in range(len(link)):
            d2 = (cen[:, s, None, 0] - obs[None, :, 0]).square_()
            for k in (1, 2):
                d2 += (cen[:, s, None, k] - obs[None, :, k]).square_()
            env = torch.minimum(env, (d2.sqrt_() - obs[None, :, 3]).min(1).values - rad[s])
        pairs = torch.from_numpy(np.asarray(data["self_pairs"], np.int64)).to(DEV)
        if len(pairs):
            a, b = pairs[:, 0], pairs[:, 1]
            d = (cen[:, a] - cen[:, b]).square().sum(-1).sqrt() - rad[a] - rad[b]
            own = torch.minimum(own, d.min(1).values)
    if len(data.get("box_link", ())):
        bl = torch.from_numpy(np.asarray(data["box_link"], np.int64)).to(DEV)
        pose, half = f("box_pose"), f("box_half")
        bc = p[:, bl] + (R[:, bl] @ pose[:, :3, None])[..., 0]
        bR = R[:, bl] @ pose[:, 3:].reshape(-1, 3, 3)
        for i, j in np.asarray(data["box_pairs"]):
            own = torch.minimum(own, _separation(bR[:, i], bc[:, i], half[i], bR[:, j], bc[:, j], half[j]))
        eb = f("env_boxes")
        for k in range(len(bl)):
            sd = _box_excess(bR[:, k, None], bc[:, k, None], half[k], obs[None, :, :3]) - obs[None, :, 3]
            env = torch.minimum(env, sd.min(1).values)
            for e in eb:
                env = torch.minimum(env, _separation(bR[:, k], bc[:, k], half[k], e[3:12].reshape(3, 3), e[:3], e[12:]))
    return torch.minimum(env, own), own


def _screen(weights, q, hidden):
    """The screen's output for rows q from its flat parameters."""
    D, H = q.shape[1], hidden
    at, parts = 0, []
    for shape in ((H, D), (H,), (H, H), (H,), (H, H), (H,), (1, H), (1,)):
        k = int(np.prod(shape))
        parts.append(weights[at:at + k].reshape(shape))
        at += k
    x = q / math.pi
    for i in range(0, 6, 2):
        x = torch.nn.functional.silu(x @ parts[i].t() + parts[i + 1])
    return (x @ parts[6].t() + parts[7])[:, 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "check" and case["mode"] == "sd":
        data, q, obs = _check_inputs(case, seed)
        obs = obs.double()
        step = max(1, (1 << 27) // max(len(obs), 3 * len(data["self_pairs"]), 512))
        got = [_distances(data, q[i:i + step].double(), obs) for i in range(0, len(q), step)]
        return None, torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])
    if kind in ("predict", "grad"):
        # the parameters a screen of this seed is created with
        data = workloads.load(ARMS["arm7"])
        ctx = ezo.Context(0)
        w = _cuda(ezo.Surrogate(ctx, data["dof"], hidden=case["hidden"], seed=int(seed)).get_params()).double()
        q = _uniform_q(data, case["n"], _generator(seed))
        if kind == "predict":
            return torch.cat([_screen(w, x.double(), case["hidden"]) for x in q.split(1 << 17)])
        tp = ezo.make_train_params()
        w.requires_grad_(True)
        t = _screen_targets(q).double().clamp(tp.clip_lo, tp.clip_hi)
        loss = torch.nn.functional.huber_loss(_screen(w, q.double(), case["hidden"]), t, delta=tp.huber_delta)
        loss.backward()
        return dict(loss=float(loss), grad=w.grad)
    return None
