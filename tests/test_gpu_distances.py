"""Signed distances of large batches (the distance field and the part bounds)
against the all-pairs kernel: the same FP32 minima bit for bit, so the small
calls that still test all pairs serve as the reference (they are checked
against the oracle elsewhere).  Scenes inside, around and far from the field's
box, more obstacles near a cell than its list holds, coordinates that are not
numbers, infinite radii, single-sided outputs, the strided layout and the
fixed-scratch call."""
import numpy as np
import pytest

import workloads
from workloads import draw

from gpu_common import load, print_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PAIRS = 1.0e8          # pairs from which a call takes the field


@pytest.fixture(scope="module")
def ezo():
    import paper_2504_10783_amd as ezo
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return ezo


@pytest.fixture(scope="module")
def ctx(ezo):
    ctx = ezo.Context(0)
    ctx.set_autotune(False)
    return ctx


def check(ezo, ctx, rob, obs, q, sd=True, own=True, **how):
    n = how.get("n") or q.shape[0]
    out = [torch.full((n,), 7, dtype=torch.uint8, device="cuda"), torch.full((n,), 99.0, device="cuda") if sd else None,
           torch.full((n,), 99.0, device="cuda") if own else None]
    ezo.check_collisions(ctx, rob, obs, q, *out, **how)
    torch.cuda.synchronize()
    return out


def scene(name, n_obs, kind):
    rng = draw.rng_for(1000 + n_obs)
    lo, hi, r = {"near": ((0.3, -0.5, 0.0), (1.3, 0.5, 1.0), 0.08), "far": ((40.0, 3.0, -9.0), (41.0, 4.0, -8.0), 0.3),
                 "dense": ((0.5, 0.0, 0.2), (0.52, 0.02, 0.22), 0.02), "flat": ((-1.5, -1.5, 0.0), (1.5, 1.5, 0.0), 0.15),
                 "bad": ((0.3, -0.5, 0.0), (1.3, 0.5, 1.0), 0.08)}[kind]
    obs = draw.obstacle_candidates(rng, n_obs, lo, hi, 0.01, r).reshape(-1, 4)
    if kind == "bad":
        obs[1, 0] = np.nan
        obs[2, 3] = np.nan
        obs[3, 3] = -0.5
    return torch.from_numpy(obs).cuda()


@pytest.mark.parametrize("name,n_obs,kind", [
    ("dof7", 40, "near"), ("dof7", 4096, "near"), ("dof7", 300, "far"), ("dof7", 700, "dense"), ("dof7", 50, "bad"),
    ("tiny", 500, "flat"), ("boxes", 194, "near"), ("forest", 3000, "near"),
    ("dof7", 0, "near"), ("boxes", 0, "near")])
def test_field_equals_all_pairs(ezo, ctx, name, n_obs, kind):
    data, desc = load(name)
    rob = ezo.Robot(ctx, desc)
    size = rob.n_spheres + rob.n_boxes
    n = 20011 if n_obs == 0 else int(PAIRS / (size * n_obs)) + 4099
    small = 4096 if n_obs == 0 else max(64, int(0.9 * PAIRS / (size * n_obs)))
    print_case("field", name, n_obs, kind, n)
    obs = scene(name, n_obs, kind)
    q = torch.from_numpy(draw.uniform_q(61, n, data["q_lo"], data["q_hi"])).cuda()
    q[5, 0], q[6, -1] = float("nan"), float("inf")
    try:
        if name == "boxes":
            ctx.set_obstacle_boxes(data["env_boxes"])
        got = check(ezo, ctx, rob, obs, q)
        if n_obs == 0:                                   # all pairs: with one obstacle out of reach of everything
            obs = torch.tensor([[1e6, 0.0, 0.0, 0.01]], device="cuda")
            small = min(small, int(0.9 * PAIRS / size))
        lo = 0
        while lo < min(n, 3 * small):
            part = q[lo:lo + small].contiguous()
            want = check(ezo, ctx, rob, obs, part)
            if n_obs == 0 and name != "boxes":           # the distant obstacle's own value
                want[1] = want[2]
            m = len(part)
            for k, (a, b) in enumerate(zip(got, want)):
                if n_obs == 0 and k != 2 and name == "boxes":
                    continue                             # the table against a frame shifted by the distant obstacle
                if n_obs == 0:
                    assert torch.allclose(a[lo:lo + m].float(), b.float(), atol=0.2, equal_nan=True) or k == 0
                    continue
                same = (a[lo:lo + m] == b) | (a[lo:lo + m].isnan() & b.isnan())
                assert bool(same.all()), (k, lo, int((~same).sum()))
            lo += small
        if n_obs > 0:
            # one output each, the strided layout, the fixed scratch
            for how in (dict(own=False), dict(sd=False)):
                one = check(ezo, ctx, rob, obs, q, **how)
                for a, b in zip(one, got):
                    assert a is None or torch.equal(a.nan_to_num(5.0) if a.is_floating_point() else a,
                                                    b.nan_to_num(5.0) if b.is_floating_point() else b)
            col = check(ezo, ctx, rob, obs, q.t().contiguous(), n=n, stride_n=1, stride_d=n, noalloc=n_obs <= 4096)
            for a, b in zip(col, got):
                assert torch.equal(a, b)
    finally:
        ctx.set_obstacle_boxes(None)


# ---- scenes and robots at the field's own edges ------------------------------

def field_scene(kind, n_obs, seed=0):
    """Obstacles about a 1 m arm: spread out; one far away, or a ground sphere of
    100 m, among them; heaped on one another; some on a point; a radius or a
    coordinate that is infinite."""
    rng = draw.rng_for(4000 + n_obs + seed)
    obs = draw.obstacle_candidates(rng, n_obs, (0.3, -0.5, 0.0), (1.3, 0.5, 1.0), 0.01, 0.06).reshape(-1, 4)
    if kind == "outlier":
        obs[1, :3] = (300.0, -40.0, 2.0)
    if kind == "ground":
        obs[1] = (0.3, 0.1, -100.3, 100.0)
    if kind == "heap":
        obs[:, :3] = np.float32([0.6, 0.0, 0.5]) + np.float32(0.02) * rng.random((n_obs, 3), dtype=np.float32)
    if kind == "point":
        obs[: n_obs // 2] = (0.5, 0.1, 0.4, 0.05)
    if kind == "inf radius":
        obs[4, 3] = np.inf
    if kind == "inf centre":
        obs[4, 1] = -np.inf
    if kind == "behind":
        obs[:, 0] += 30.0
    return obs


def field_against_pairs(ezo, ctx, rob, desc, obs, q):
    """A batch that the field takes (its tuning entry says so) against calls of 64
    rows of it, which test all pairs: the same values, rows of its start and end."""
    n, o = len(q), torch.from_numpy(np.ascontiguousarray(obs)).cuda()
    ezo.tune_cache_clear()
    ctx.set_autotune(True)
    try:
        got = check(ezo, ctx, rob, o, q)
        assert [e.get("field") for e in ezo.tune_cache_entries() if e["kernel"] == "check_sd"] == [1]
    finally:
        ctx.set_autotune(False)
        ezo.tune_cache_clear()
    untuned = check(ezo, ctx, rob, o, q)
    for a, b in zip(untuned, got):
        assert torch.equal(a, b)
    for lo in [*range(0, 640, 64), n - 64]:
        want = check(ezo, ctx, rob, o, q[lo:lo + 64].contiguous())
        for k, (a, b) in enumerate(zip(got, want)):
            same = (a[lo:lo + 64] == b) | (a[lo:lo + 64].isnan() & b.isnan())
            assert bool(same.all()), (k, lo, int((~same).sum()))
    return got


@pytest.mark.parametrize("kind,n_obs,n", [
    ("spread", 600, 4000), ("outlier", 600, 4000), ("ground", 600, 4000), ("heap", 3000, 2000), ("point", 3000, 2000),
    ("inf radius", 600, 4000), ("inf centre", 600, 4000), ("behind", 600, 4000), ("spread", 6000, 6000),
    ("heap", 200, 20000), ("spread", 129, 20000)])
def test_field_scenes(ezo, ctx, kind, n_obs, n):
    """Cells whose list is too long, blocks of cells with more obstacles than a
    workgroup holds, and obstacles far larger or farther than the robot."""
    data, desc = load("dof7")
    rob = ezo.Robot(ctx, desc)
    print_case("field scene", kind, n_obs, n)
    q = torch.from_numpy(draw.uniform_q(4100, n, data["q_lo"], data["q_hi"])).cuda()
    q[5, 0], q[6, -1] = float("nan"), float("inf")
    field_against_pairs(ezo, ctx, rob, desc, field_scene(kind, n_obs), q)


@pytest.mark.parametrize("dof,per_link,prismatic,n", [(1, 1, False, 1 << 20), (5, 16, True, 8000), (8, 128, False, 2000)])
def test_field_robots(ezo, ctx, dof, per_link, prismatic, n):
    """The smallest and the largest robot (1024 spheres, every part pair), and
    sliding joints far beyond their limits, where no bound of the field holds."""
    desc = draw.arm_dh(draw.rng_for(4200 + dof), dof, per_link)
    if prismatic:
        desc["joint_type"] = (np.arange(dof) % 3 == 1).astype(np.int32)
    if per_link == 128:
        s = np.arange(1024).reshape(16, 64)                # [part][sphere]
        desc["self_pairs"] = np.array([(s[a, i], s[b, 1 + i]) for a in range(16) for b in range(a, 16) for i in range(3)], np.int32)
    print_case("field robot", dof, per_link, prismatic, n)
    q = draw.uniform_q(4300, n, desc["q_lo"], desc["q_hi"])
    if prismatic:
        q[::3] *= np.where(desc["joint_type"] == 1, 40.0, 1.0).astype(np.float32)
    rob = ezo.Robot(ctx, desc)
    field_against_pairs(ezo, ctx, rob, desc, field_scene("outlier", 700), torch.from_numpy(q).cuda())


def test_field_without_obstacles(ezo, ctx):
    """Self distances of a batch past the field's line, against the oracle."""
    import oracle
    from gpu_common import BAND, SD_TOL
    data, desc = load("dof7")
    rob, orob = ezo.Robot(ctx, desc), oracle.Robot(desc)
    n, m = 100_003, 2000
    print_case("field without obstacles", n)
    q = draw.uniform_q(4400, n, data["q_lo"], data["q_hi"])
    flags, sd, own = check(ezo, ctx, rob, torch.zeros((0, 4), device="cuda"), torch.from_numpy(q).cuda())
    assert torch.equal(sd, own) and torch.equal(flags, (own < 0).to(torch.uint8))
    fo, so, *_ = oracle.check(orob, np.zeros((0, 4)), q[:m].astype(np.float64))
    assert np.abs(own[:m].cpu().numpy() - so).max() <= SD_TOL
    sure = np.abs(so) >= BAND
    assert np.array_equal(flags[:m].cpu().numpy()[sure], fo[sure])


@pytest.mark.parametrize("name,n_obs,n,field", [
    ("dof7", 4, 400_000, 0), ("dof7", 16, 100_000, 0), ("tiny", 20, 1 << 20, 0), ("dof7", 65535, 30, 0),
    ("dof7", 16384, 200, 0), ("dof7", 0, 20_000, 0), ("forest", 15, 1 << 20, 0),
    ("dof7", 128, 30_000, 1), ("dof7", 512, 5600, 1), ("dof7", 4096, 700, 1), ("tiny", 300, 300_000, 1)])
def test_kernel_by_size(ezo, ctx, name, n_obs, n, field):
    """All pairs where there is little to leave out or the field's build would cost
    more than the batch (few obstacles, few spheres, few configurations among very
    many obstacles), the field where it saves."""
    data, desc = load(name)
    rob = ezo.Robot(ctx, desc)
    print_case("kernel by size", name, n_obs, n)
    obs = torch.from_numpy(field_scene("spread", max(n_obs, 1))[:n_obs].copy()).cuda()
    q = torch.from_numpy(draw.uniform_q(4500, n, data["q_lo"], data["q_hi"])).cuda()
    ezo.tune_cache_clear()
    ctx.set_autotune(True)
    try:
        check(ezo, ctx, rob, obs, q)
        assert [e.get("field", 0) for e in ezo.tune_cache_entries() if e["kernel"] == "check_sd"] == [field]
    finally:
        ctx.set_autotune(False)
        ezo.tune_cache_clear()
