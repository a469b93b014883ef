"""The BVH walks on rays that decide their box tests by a hair, bit for bit against the oracle
trying every triangle: directions with zero and negative-zero components, origins on the scene's
planes, origins 10^5 and 10^7 m away, a walk that spills its stack, dynamic triangles whose
common box the rays meet, graze or miss."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


def _layers():
    """2,000 large triangles one behind the other along z, each covering half of the same square"""
    n = 2000
    rng = np.random.default_rng(9)
    z = np.linspace(1.0, 50.0, n)[:, None]
    corner = rng.integers(0, 4, n)
    sq = np.array([[-5.0, -5.0], [5.0, -5.0], [5.0, 5.0], [-5.0, 5.0]])
    v = np.zeros((n, 3, 3))
    for k in range(3):
        v[:, k, :2] = sq[(corner + k) % 4]
    v[:, :, 2] = z + rng.uniform(-0.01, 0.01, (n, 3))
    return I.Scene("layers", v.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.uint32).reshape(-1, 3),
                   np.zeros(n, np.uint32), np.array([[0.5, 0.5, 0.5, 0.0, 0.0, 0.0]], np.float32))


def _rays(kind, scene):
    rng = np.random.default_rng(4)
    n = 3000
    lo, hi = scene.verts.min(0), scene.verts.max(0)
    o = rng.uniform(lo, hi, (n, 3)).astype(np.float32)
    if kind == "axis":
        d = rng.choice(np.array([-1.0, -0.0, 0.0, 1.0], np.float32), (n, 3))
        d[(d == 0).all(1)] = (0.0, -0.0, -1.0)
        d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
        for a in range(3):                          # half of the origins share a coordinate with a vertex
            on = rng.random(n) < 0.5
            o[on, a] = scene.verts[rng.integers(0, len(scene.verts), int(on.sum())), a]
        return o, d
    if kind == "far":
        d = rng.normal(size=(n, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        d = d.astype(np.float32)
        dist = np.where(np.arange(n) % 2, 1e5, 1e7).astype(np.float32)[:, None]
        return o - dist * d, d
    if kind == "layers":
        o[:, 2] = rng.uniform(-1.0, 51.0, n)
        d = rng.normal(size=(n, 3)) * (0.02, 0.02, 1.0)
        return o, (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    return o, I.random_rays(n, lo, hi, seed=12)[1]


@pytest.mark.parametrize("kind", ["axis", "far", "layers", "dynamic"])
def test_walks_equal_brute_force(kind):
    scene = _layers() if kind == "layers" else I.room_scene()
    ctx = gi.Context(width=64, height=64)
    ctx.build_bvh(scene)
    osc = O.OracleScene(scene, use_bvh=False)
    if kind == "layers":
        assert 3 * int(ctx.dims()[10]) + 1 > 16, "the walk must spill past the LDS part of the stack"
    if kind == "dynamic":
        # three triangles of one box, one of them flat in it
        tv = np.array([[1, 1, 1, 2, 1, 1, 1, 2, 1], [2, 1.5, 2, 2, 2, 2, 2.5, 1.5, 2.5],
                       [1, 2, 1, 1, 2, 2.5, 2.5, 2, 1]], np.float32)
        mats = np.zeros(3, np.uint32)
        ctx.set_dynamic(tv, mats)
        osc.set_dynamic(tv, mats)
    o, d = _rays(kind, scene)
    n = len(o)
    if kind == "dynamic":
        d[: n // 3] = tv[1, :3] - o[: n // 3]       # a third of the rays through a vertex, not unit length
    o4 = np.full((n, 4), 3.0e38, np.float32)
    o4[:, :3] = o
    d4 = np.zeros((n, 4), np.float32)
    d4[:, :3] = d
    tri = torch.zeros(n, dtype=torch.int32, device="cuda")
    t = torch.zeros(n, dtype=torch.float32, device="cuda")
    ctx.trace_rays(torch.from_numpy(o4).cuda(), torch.from_numpy(d4).cuda(), tri, t)
    otri, ot = osc.closest(o, d)
    assert (otri != 0xFFFFFFFF).mean() > 0.1
    assert np.array_equal(tri.cpu().numpy().view(np.uint32), otri)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), ot.view(np.uint32))
    # segments that end just before, at and just after the closest hit
    tm = (np.where(otri != 0xFFFFFFFF, ot, 5.0) * np.array([0.999, 1.0, 1.001], np.float32)[np.arange(n) % 3]).astype(np.float32)
    o4[:, 3] = tm
    ctx.trace_rays(torch.from_numpy(o4).cuda(), torch.from_numpy(d4).cuda(), tri, t, any_hit=True)
    assert np.array_equal(tri.cpu().numpy().view(np.uint32), osc.any(o, d, tm))


@pytest.mark.parametrize("width,height,rays", [(8, 8, 1), (488, 8, 64), (488, 16, 64), (976, 8, 63)])
def test_every_block_of_probe_rays_is_traced(width, height, rays):
    """1, 61 and 122 blocks of rays (fewer, about as many and more than the hit list's stripes) and
    a part of a block at the end: every ray record and cell sum against the oracle"""
    _run_stage_parity(I.room_scene(), dict(width=width, height=height, rays_per_probe=rays, table_log2=16), [0, 1])
