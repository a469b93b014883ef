"""Moving triangles are tested behind their common box: rays along its faces and rays of tiny
directions (components below 1e-30, whose reciprocals are cut off) must not lose a hit.  Bit for bit
against the oracle, which has no box."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402


def _quad(axis, side):
    """[side - 1, side] along `axis` (0 is a face), [-1, 1] along the next, 0 along the last: [2, 9]"""
    v = np.zeros((4, 3), np.float32)
    v[:, axis] = np.array([-1, -1, 0, 0], np.float32) + side
    v[:, (axis + 1) % 3] = (-1, 1, 1, -1)
    return v[[0, 1, 2, 0, 2, 3]].reshape(2, 9)


@pytest.mark.parametrize("rays", ["face", "tiny"])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_box_keeps_every_hit(axis, side, rays):
    scene = I.room_scene()
    far = I.Scene("room", scene.verts + np.float32(100.0), scene.idx, scene.tri_mat, scene.materials)
    ctx = gi.Context(width=64, height=64)
    ctx.build_bvh(far)
    osc = O.OracleScene(far, use_bvh=False)
    tv = _quad(axis, side)
    ctx.set_dynamic(tv, np.zeros(2, np.uint32))
    osc.set_dynamic(tv, np.zeros(2, np.uint32))
    b, c = (axis + 1) % 3, (axis + 2) % 3
    n = 512
    rng = np.random.default_rng(axis + 3 * side)
    o = np.zeros((n, 3), np.float32)
    d = np.zeros((n, 3), np.float32)
    o[:, b] = rng.uniform(-0.9, 0.9, n)
    o[:, c] = rng.choice([-5.0, 5.0], n)
    if rays == "face":          # in the plane of the box's face at 0, straight at the quad's edge
        d[:, c] = -np.sign(o[:, c])
        d[:, axis] = rng.choice([0.0, -0.0], n)
    else:
        at = np.zeros((n, 3), np.float32)
        at[:, axis] = side - rng.uniform(0.1, 0.9, n)
        at[:, b] = rng.uniform(-0.9, 0.9, n)
        d = (at - o) * np.float32(1e-31)
    o4 = np.full((n, 4), 3.0e38, np.float32)
    o4[:, :3] = o
    d4 = np.zeros((n, 4), np.float32)
    d4[:, :3] = d
    tri = torch.zeros(n, dtype=torch.int32, device="cuda")
    t = torch.zeros(n, dtype=torch.float32, device="cuda")
    to, td = torch.from_numpy(o4).cuda(), torch.from_numpy(d4).cuda()
    ctx.trace_rays(to, td, tri, t)
    otri, ot = osc.closest(o, d)
    assert (otri != 0xFFFFFFFF).mean() > 0.9
    assert np.array_equal(tri.cpu().numpy().view(np.uint32), otri)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), ot.view(np.uint32))
    ctx.trace_rays(to, td, tri, t, any_hit=True)
    assert np.array_equal(tri.cpu().numpy().view(np.uint32), (otri != 0xFFFFFFFF).astype(np.uint32))
    ctx.close()
