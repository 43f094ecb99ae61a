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
