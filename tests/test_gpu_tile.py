"""GPU checks of the flags tile at the edges of its ranges: batch sizes around
the tiles and the eight lanes of a configuration, joint counts from 1 to 8,
obstacle counts around the grid sizes (none, one, past the 16-bit lists),
cells whose state is a certain hit, robots without spheres on some links; and
the bisection's levels per round, which change with the number of candidates
in the call's list and must not change a result."""
import json

import numpy as np
import pytest

import oracle
from workloads import draw

from gpu_common import BAND, load, print_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ezo():
    import paper_2504_10783_amd as ezo
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return ezo


@pytest.fixture(scope="module")
def ctx(ezo):
    return ezo.Context(0)


def arm(dof, per_link, seed, prismatic=False):
    rng = draw.rng_for(seed)
    d = draw.arm_dh(rng, dof, per_link)
    keep = np.arange(len(d["sphere_link"]))
    if dof > 2:                                        # a link without spheres
        keep = keep[d["sphere_link"] != 1]
    for k in ("sphere_link", "sphere_xyz", "sphere_r"):
        d[k] = d[k][keep]
    d["self_pairs"] = draw.self_pair_candidates(d["sphere_link"])
    if prismatic:
        d["joint_type"] = (np.arange(dof) % 3 == 1).astype(np.int32)
    return d


@pytest.mark.parametrize("dof,per_link,n_obs,n,prismatic", [
    (1, 1, 1, 1, False), (2, 3, 31, 7, True), (3, 5, 32, 9, False), (5, 16, 255, 63, True), (7, 10, 256, 65, False),
    (7, 10, 70000, 33, False), (8, 64, 300, 129, True), (7, 10, 0, 64, False)])
def test_flags_at_tile_edges(ezo, ctx, dof, per_link, n_obs, n, prismatic):
    print_case("tile edges", dof, per_link, n_obs, n, prismatic)
    desc = arm(dof, per_link, 900 + dof, prismatic)
    rng = draw.rng_for(7 * n_obs + n)
    # radii up to several cells: cells that lie inside an obstacle
    obs = draw.obstacle_candidates(rng, n_obs, (-1.0, -1.0, -0.5), (1.2, 1.0, 1.0), 0.002, 0.004) if n_obs > 60000 else \
        draw.obstacle_candidates(rng, n_obs, (-1.0, -1.0, -0.5), (1.2, 1.0, 1.0), 0.01, 0.25 if n_obs < 60 else 0.09)
    obs = obs.reshape(-1, 4)
    q = draw.uniform_q(41 + n, n, desc["q_lo"], desc["q_hi"])
    rob, orob = ezo.Robot(ctx, desc), oracle.Robot(desc)
    fo, sd, *_ = oracle.check(orob, obs.astype(np.float64), q.astype(np.float64))
    flags = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    ezo.check_collisions(ctx, rob, torch.from_numpy(obs).cuda(), torch.from_numpy(q).cuda(), flags)
    got = flags.cpu().numpy()
    out = np.abs(sd) >= BAND
    assert np.array_equal(got[out], fo[out])


@pytest.mark.parametrize("pairs", ["none", "one", "few", "some", "all", "boxes", "boxes too"])
@pytest.mark.parametrize("dof", range(1, 9))
def test_flags_by_joints_and_pairs(ezo, ctx, dof, pairs):
    """A record's size goes by the joints and by whether there are self pairs of
    spheres; the lanes an overlapping pair of link parts takes by the number of its
    pairs (1 to 64 a pair of parts here); a robot of boxes keeps no lists,
    and one with boxes no cell states."""
    n = 199
    desc = arm(dof, 16 if pairs != "one" else 2, 700 + dof, dof % 2 == 0)
    p = np.asarray(desc["self_pairs"], np.int32).reshape(-1, 2)
    rng = draw.rng_for(710 + dof)
    if pairs in ("none", "boxes"):
        p = p[:0]
    elif pairs in ("few", "some") and len(p):
        p = p[np.sort(rng.choice(len(p), len(p) // (20 if pairs == "few" else 10), replace=False))]
    desc["self_pairs"] = p
    if pairs == "boxes":
        for k in ("sphere_link", "sphere_xyz", "sphere_r"):
            desc[k] = desc[k][:0]
    if pairs.startswith("boxes"):
        desc["box_link"] = np.arange(dof, dtype=np.int32)
        desc["box_pose"] = np.tile(np.concatenate([np.zeros(3), np.eye(3).ravel()]), (dof, 1))
        desc["box_half"] = rng.uniform(0.03, 0.12, (dof, 3))
        desc["box_pairs"] = np.array([(i, j) for i in range(dof) for j in range(i + 2, dof)], np.int32).reshape(-1, 2)
    print_case("joints and pairs", dof, pairs, len(desc["self_pairs"]))
    obs = draw.obstacle_candidates(rng, 40, (-1.0, -1.0, -0.5), (1.2, 1.0, 1.0), 0.02, 0.06).reshape(-1, 4)
    q = draw.uniform_q(720 + dof, n, desc["q_lo"], desc["q_hi"])
    rob, orob = ezo.Robot(ctx, desc), oracle.Robot(desc)
    ot, qt = torch.from_numpy(obs).cuda(), torch.from_numpy(q).cuda()
    fo, sd, *_ = oracle.check(orob, obs.astype(np.float64), q.astype(np.float64))
    sure = np.abs(sd) >= BAND
    size = dict(arch=torch.cuda.get_device_properties(0).gcnArchName.split(":")[0], kernel="check_flags", dof=dof,
                spheres=rob.n_spheres, self_pairs=rob.n_self, boxes=rob.n_boxes, obstacles=len(obs), log2_items=7)
    ctx.set_autotune(False)
    try:
        for T, W in ((0, 0), (64, 8), (64, 1), (8, 2), (4, 8)):
            ezo.tune_cache_clear()
            if T:
                assert ezo.tune_cache_import(json.dumps(dict(size, T=T, W=W, stage=0, depth=1, us=0.0),
                                                        separators=(",", ":"))) == 1
            flags = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
            ezo.check_collisions(ctx, rob, ot, qt, flags)
            assert np.array_equal(flags.cpu().numpy()[sure], fo[sure]), (T, W)
    finally:
        ctx.set_autotune(True)
        ezo.tune_cache_clear()


def test_bisection_levels_give_identical_results(ezo, ctx):
    """Three edges with 0, 1 and many candidates in one call (one level per
    round), against calls of a few candidates each (more levels): the same
    bits.  The tile takes candidates of several edges."""
    data, desc = load("dof7")
    rob = ezo.Robot(ctx, desc)
    obs = torch.from_numpy(data["obstacles"]).cuda()
    pool = torch.from_numpy(draw.uniform_q(77, 40000, data["q_lo"], data["q_hi"])).cuda()
    fl = torch.empty(len(pool), dtype=torch.uint8, device="cuda")
    ezo.check_collisions(ctx, rob, obs, pool, fl)
    cand = pool[fl.bool()][:9001]
    n = len(cand)
    print_case("bisection levels", n)
    v1 = torch.from_numpy(data["edges"][0, :1]).cuda()
    edges = torch.stack([v1.repeat(2, 1), torch.from_numpy(data["edges"][0]).cuda(),
                         torch.from_numpy(data["edges"][0]).cuda().flip(0)]).contiguous()

    def run(counts, S, cap):
        E = len(counts)
        ci = torch.arange(cap, dtype=torch.int32, device="cuda").repeat(E, 1).contiguous()
        nc = torch.tensor(counts, dtype=torch.int32, device="cuda")
        out = (torch.full((E, 7, cap), -7.0, device="cuda"), torch.full((E, 7, cap), -7.0, device="cuda"),
               torch.full((E, cap), -7.0, device="cuda"), torch.full((E, cap), 9, dtype=torch.uint8, device="cuda"))
        ezo.project_bisect(ctx, rob, obs, edges[3 - E:].contiguous(), S, ci, nc, 11, *out)
        torch.cuda.synchronize()
        return out

    S = cand.t().contiguous().view(1, 7, n)
    ctx.set_autotune(False)
    try:
        big = run([0, 1, n], S.repeat(3, 1, 1).contiguous(), n)
        assert bool((big[2][0] == -7.0).all()) and bool((big[2][1, 1:] == -7.0).all())
        for lo, m in ((0, 1), (1, 5), (100, 700), (2000, 2500)):
            small = run([m], S[:, :, lo:lo + m].contiguous(), m)
            for a, b in zip(small, big):
                assert torch.equal(a[0], b[2][..., lo:lo + m]), (lo, m)
    finally:
        ctx.set_autotune(True)


def test_bisection_over_several_candidate_lists(ezo, ctx):
    """So many edges x candidate slots that the candidates come in two lists (4800 x
    57 344): edges of both and of their ends, against a call with those edges only."""
    desc = arm(2, 3, 77)
    rob = ezo.Robot(ctx, desc)
    rng = draw.rng_for(78)
    obs = torch.from_numpy(draw.obstacle_candidates(rng, 20, (-0.6, -0.6, -0.2), (0.6, 0.6, 0.2), 0.05, 0.15).reshape(-1, 4)).cuda()
    E, cap, stride, group = 4800, 57344, 64, (1 << 28) // 57344
    assert group < E < 2 * group
    print_case("two candidate lists", E, cap)
    S = torch.from_numpy(draw.uniform_q(79, E * stride, desc["q_lo"], desc["q_hi"])).cuda().view(E, stride, 2).transpose(1, 2).contiguous()
    edges = torch.from_numpy(draw.uniform_q(80, 2 * E, desc["q_lo"], desc["q_hi"])).cuda().view(E, 2, 2).contiguous()
    some = torch.tensor([0, 3, group - 1, group, group + 1, E - 1], device="cuda")

    def run(ids, capacity):
        n = len(ids)
        nc = torch.zeros(n, dtype=torch.int32, device="cuda")
        nc[torch.isin(ids, some)] = torch.tensor([1, 64, 7, 40, 64, 33], dtype=torch.int32, device="cuda")
        ci = torch.zeros((n, capacity), dtype=torch.int32, device="cuda")
        ci[:, :64] = torch.arange(64, dtype=torch.int32, device="cuda")
        out = [torch.full(s, -7.0, device="cuda") for s in ((n, 2, capacity), (n, 2, capacity), (n, capacity))]
        out.append(torch.full((n, capacity), 9, dtype=torch.uint8, device="cuda"))
        ezo.project_bisect(ctx, rob, obs, edges[ids].contiguous(), S[ids].contiguous(), ci, nc, 9, *out)
        torch.cuda.synchronize()
        return [x[torch.isin(ids, some)][..., :64].clone() for x in out] + [int((out[2] != -7.0).sum())]

    ctx.set_autotune(False)
    try:
        big = run(torch.arange(E, device="cuda"), cap)
        small = run(some, 64)
        for a, b in zip(big, small):
            assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b
        assert big[-1] == 1 + 64 + 7 + 40 + 64 + 33
    finally:
        ctx.set_autotune(True)
        torch.cuda.empty_cache()


def test_largest_robot_with_every_part_pair(ezo, ctx):
    """Every part pair a block (136 with eight links), 1024 spheres, 64 boxes:
    the bisection's smallest tile passes 64 KB of LDS and is still accepted."""
    rng = draw.rng_for(5)
    desc = draw.arm_dh(rng, 8, 128)
    s = np.arange(1024).reshape(16, 64)                # [part][sphere]
    desc["self_pairs"] = np.array([(s[a, 0], s[b, 1]) for a in range(16) for b in range(a, 16)], np.int32)
    desc["box_link"], desc["box_pose"], desc["box_half"] = (np.concatenate([x] * 6)[:64] for x in
                                                            draw.arm_boxes(rng, desc, 12))
    desc["box_half"] = desc["box_half"] * np.float32(0.2)
    desc["box_pairs"] = np.zeros((0, 2), np.int32)
    rob, orob = ezo.Robot(ctx, desc), oracle.Robot(desc)
    obs = draw.obstacle_candidates(rng, 40, (-1.5, -1.5, -1.0), (1.5, 1.5, 1.5), 0.02, 0.05)
    q = draw.uniform_q(3, 21, desc["q_lo"], desc["q_hi"])
    print_case("largest robot, every part pair")
    fo, sd, *_ = oracle.check(orob, obs.astype(np.float64), q.astype(np.float64))
    ot, qt = torch.from_numpy(obs).cuda(), torch.from_numpy(q).cuda()
    flags = torch.empty(len(q), dtype=torch.uint8, device="cuda")
    ctx.set_autotune(False)
    try:
        ezo.check_collisions(ctx, rob, ot, qt, flags)
        out = np.abs(sd) >= BAND
        assert np.array_equal(flags.cpu().numpy()[out], fo[out])
        n = len(q)
        ci = torch.arange(n, dtype=torch.int32, device="cuda").view(1, n)
        res = (torch.empty((1, 8, n), device="cuda"), torch.empty((1, 8, n), device="cuda"),
               torch.empty((1, n), device="cuda"), torch.empty((1, n), dtype=torch.uint8, device="cuda"))
        edges = torch.stack([qt[0], qt[0]]).view(1, 2, 8).contiguous()      # L = one point: the projection
        ezo.project_bisect(ctx, rob, ot, edges, qt.t().contiguous().view(1, 8, n), ci,
                           torch.tensor([n], dtype=torch.int32, device="cuda"), 0, *res)
        assert torch.equal(res[0][0].t(), qt)           # no bisection step: c* = c
        if out[0]:
            assert bool((res[3] == int(fo[0])).all())
    finally:
        ctx.set_autotune(True)


@pytest.mark.parametrize("n_obs", [1, 31, 32, 255, 256, 1023, 1025, 2500])
@pytest.mark.parametrize("kind", ["near", "far", "bad"])
def test_grid_of_any_scene_equals_all_pairs(ezo, ctx, n_obs, kind):
    """Every grid size and obstacle counts around a chunk of the grid's build: the
    flags sweep against the all-pairs distances' own flags, which use no grid."""
    data, desc = load("dof7")
    rob = ezo.Robot(ctx, desc)
    rng = draw.rng_for(7000 + n_obs)
    lo, hi = ((0.3, -0.6, 0.0), (1.3, 0.6, 1.0)) if kind != "far" else ((0.9, 3.0, -9.0), (41.0, 4.0, 0.2))
    obs = draw.obstacle_candidates(rng, n_obs, lo, hi, 0.01, 0.06).reshape(-1, 4)
    if kind == "bad" and n_obs > 3:
        obs[1, 0], obs[2, 3] = np.nan, np.nan        # (a radius below zero has no distance to compare: the sweep squares it)
    n = 300
    q = torch.from_numpy(draw.uniform_q(7001, n, data["q_lo"], data["q_hi"])).cuda()
    o = torch.from_numpy(obs).cuda()
    print_case("grid", kind, n_obs)
    flags = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    ezo.check_collisions(ctx, rob, o, q, flags)
    want = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
    sd = torch.zeros(n, device="cuda")
    ezo.check_collisions(ctx, rob, o, q, want, sd)
    torch.cuda.synchronize()
    sure = sd.abs() > 1e-5                                   # (a square root apart)
    assert torch.equal(flags[sure], want[sure]) and int(sure.sum()) > n - 5
