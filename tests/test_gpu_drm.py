"""GPU parity of the DRM collision map (appendix, DRM construction) against
the oracle's plain definition: every (voxel, node) bit equal wherever the
oracle's signed distance lies outside +-1e-5 m (the map tests robot spheres
and boxes against voxel spheres: exact distances, no box-box axes), on the whole grid for the 3-DOF arm and on a dense block plus
random voxels for the 7-DOF sphere and box arms; id lists equal the bitset
rows; ragged node counts, padded rows and empty inputs."""
import numpy as np
import pytest

import oracle
from workloads import draw

from gpu_common import BAND, f32_up, load, print_case

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


def unpack(cmap, n):
    """bool [V][n] from the int32 bitset rows."""
    w = cmap.cpu().numpy().view(np.uint32)
    bits = np.unpackbits(w.view(np.uint8), axis=1, bitorder="little")
    return bits[:, :n].astype(bool), bits[:, n:]


def check_rows(got, voxels, desc, q, lo, side, dims, band, label):
    hits, sd = oracle.collision_map(oracle.Robot(desc), f32_up(q), f32_up(lo), float(np.float32(side)), dims, voxels)
    ok = np.abs(sd) >= band
    print(f"{label}: {len(voxels)} voxels x {len(q)} nodes, hit fraction {hits.mean():.4f}, "
          f"in band {1 - ok.mean():.2e}")
    assert np.array_equal(got[voxels][ok], hits[ok])
    return hits


def test_map_whole_grid_tiny(ezo, ctx):
    data, desc = load("tiny")
    rob = ezo.Robot(ctx, desc)
    q = draw.uniform_q(31, 301, data["q_lo"], data["q_hi"])            # ragged: 9 full words + 13 bits
    lo, side, dims = np.array([-1.6, -1.6, -0.15], np.float32), 0.1, (32, 32, 3)
    print_case("map tiny", len(q), dims)
    cmap = ezo.collision_map(ctx, rob, torch.from_numpy(q).cuda(), lo, side, dims)
    torch.cuda.synchronize()
    got, pad = unpack(cmap, len(q))
    assert not pad.any()                                             # no bit past the last node
    hits = check_rows(got, np.arange(np.prod(dims)), desc, q, lo, side, dims, BAND, "tiny")
    assert 0.001 < hits.mean() < 0.5


@pytest.mark.parametrize("name,band", [("dof7", BAND), ("boxes", BAND)])
def test_map_block_and_random_voxels(ezo, ctx, name, band):
    data, desc = load(name)
    rob = ezo.Robot(ctx, desc)
    q = draw.uniform_q(32, 2001, data["q_lo"], data["q_hi"])
    lo, side, dims = np.array([-1.3, -1.3, -0.6], np.float32), 0.1, (26, 26, 20)
    print_case("map", name, len(q), dims)
    cmap = ezo.collision_map(ctx, rob, torch.from_numpy(q).cuda(), lo, side, dims)
    torch.cuda.synchronize()
    got, pad = unpack(cmap, len(q))
    assert not pad.any()
    i, j, k = np.meshgrid(np.arange(7, 19), np.arange(7, 19), np.arange(4, 14), indexing="ij")
    block = ((k * dims[1] + j) * dims[0] + i).ravel()
    rnd = np.random.default_rng(6).choice(np.prod(dims), 400, replace=False)
    hits = check_rows(got, np.unique(np.concatenate([block, rnd])), desc, q, lo, side, dims, band, name)
    assert hits.mean() > 0.01


def test_map_lists_padding_and_empty(ezo, ctx):
    data, desc = load("dof7")
    rob = ezo.Robot(ctx, desc)
    q = torch.from_numpy(draw.uniform_q(33, 333, data["q_lo"], data["q_hi"])).cuda()
    lo, side, dims = np.array([-1.0, -1.0, -0.5], np.float32), 0.125, (16, 16, 12)
    V = int(np.prod(dims))
    # a padded row stride gives the same bits
    wide = torch.full((V, 16), -1, dtype=torch.int32, device="cuda")       # stale contents: cleared by the call
    m1 = ezo.collision_map(ctx, rob, q, lo, side, dims)
    m2 = ezo.collision_map(ctx, rob, q, lo, side, dims, out=wide)
    torch.cuda.synchronize()
    assert torch.equal(m2[:, :m1.shape[1]], m1) and not bool(m2[:, m1.shape[1]:].any())
    offsets, ids = ezo.collision_map_lists(ctx, m1, 333)
    torch.cuda.synchronize()
    got, _ = unpack(m1, 333)
    off = offsets.cpu().numpy()
    idn = ids.cpu().numpy()
    assert off[0] == 0 and off[-1] == len(idn) == got.sum()
    for v in np.random.default_rng(7).choice(V, 300, replace=False):
        assert np.array_equal(idn[off[v]:off[v + 1]], np.nonzero(got[v])[0])
    # no nodes: the map is cleared, the lists are empty
    m3 = ezo.collision_map(ctx, rob, q[:0], lo, side, dims, out=wide)
    torch.cuda.synchronize()
    assert not bool(m3.any())
    offsets, ids = ezo.collision_map_lists(ctx, m1[:, :0], 0)
    torch.cuda.synchronize()
    assert len(ids) == 0 and not bool(offsets.any())


@pytest.mark.parametrize("name,n,dims,side", [("dof7", 1, (64, 64, 40), 0.05), ("boxes", 9, (70, 60, 33), 0.05),
                                              ("dof7", 40, (9, 7, 5), 0.4), ("forest", 263, (61, 47, 37), 0.06)])
def test_map_spans_and_node_bytes(ezo, ctx, name, n, dims, side):
    """Voxels split over several workgroups (more than one table holds, or few
    nodes) and node counts around a byte of a row."""
    data, desc = load(name)
    rob = ezo.Robot(ctx, desc)
    q = draw.uniform_q(35, n, data["q_lo"], data["q_hi"])
    lo = np.array([-0.5 * d * side for d in dims], np.float32)
    print_case("map spans", name, n, dims)
    V = int(np.prod(dims))
    out = torch.full((V, (n + 31) // 32), -1, dtype=torch.int32, device="cuda")
    ezo.collision_map(ctx, rob, torch.from_numpy(q).cuda(), lo, side, dims, out=out)
    torch.cuda.synchronize()
    got, pad = unpack(out, n)
    assert not pad.any()
    parts = max(-(-V // 49152), min((512 + (n + 7) // 8 - 1) // ((n + 7) // 8), V // 4096), 1)
    span = -(-V // parts)
    edges = [v + d for v in range(0, V, span) for d in range(-40, 40)]
    near = np.argsort(-got.sum(1), kind="stable")[:300]
    voxels = np.unique(np.clip(np.concatenate([edges, near, np.random.default_rng(8).choice(V, min(V, 400), replace=False)]), 0, V - 1).astype(int))
    hits = check_rows(got, voxels, desc, q, lo, side, dims, BAND, name)
    assert hits.any()


@pytest.mark.parametrize("rows,words,density", [(1, 1, 0.5), (3, 64, 0.0), (4095, 3, 0.3), (4097, 65, 0.02),
                                                (700, 511, 0.4), (300, 1100, 0.001), (300001, 2, 0.1)])
def test_map_lists_of_any_rows(ezo, ctx, rows, words, density):
    """Row counts around the scan's tiles and chunks, words around the loads in
    flight, empty to dense rows: offsets and ids against numpy."""
    rng = np.random.default_rng(rows)
    bits = rng.random((rows, words * 32)) < density
    if rows > 2:
        bits[rows // 2] = True                                       # a full row
        bits[rows // 3] = False
    print_case("lists", rows, words, density)
    packed = np.packbits(bits, axis=1, bitorder="little").view(np.int32)
    offsets, ids = ezo.collision_map_lists(ctx, torch.from_numpy(packed.copy()).cuda(), words * 32)
    torch.cuda.synchronize()
    r, c = np.nonzero(bits)
    want = np.zeros(rows + 1, np.int64)
    np.cumsum(bits.sum(1), out=want[1:])
    assert np.array_equal(offsets.cpu().numpy(), want) and np.array_equal(ids.cpu().numpy(), c)


@pytest.mark.parametrize("name,n,dims,side", [("boxes", 17, (230, 220, 6), 0.012), ("boxes", 3, (40, 1, 900), 0.004),
                                              ("dof7", 17, (230, 220, 6), 0.012)])
def test_map_spans_of_part_of_a_plane(ezo, ctx, name, n, dims, side):
    """Planes wider than a span, and planes of one row: a box's rows over its lanes."""
    test_map_spans_and_node_bytes(ezo, ctx, name, n, dims, side)
