"""Rays whose origin along an axis times the reciprocal direction nears the largest float: the box
tests must not lose what the triangle test finds.  Bit for bit against the oracle trying every
triangle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402

# a direction component of at most 1e-30 has the reciprocal 1e30: an origin of 3.4028235e8 makes the
# largest float.  Origins on both sides of it, 32 apart (a float's step there)
ALONG = np.float32(3.4028235e8) + 32 * np.arange(-400, 400).astype(np.float32)


@pytest.mark.parametrize("moving", [False, True])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_origins_at_the_largest_reciprocal(axis, sign, moving):
    b, c = (axis + 1) % 3, (axis + 2) % 3
    # one quad across the rays, in the plane c = 0, around the origins along `axis`
    v = np.zeros((4, 3), np.float32)
    v[:, axis] = sign * np.float32(1e8) * np.array([3.3, 3.3, 3.5, 3.5], np.float32)
    v[:, b] = np.float32(1e7) * np.array([-1, 1, 1, -1], np.float32)
    f = np.array([[0, 1, 2], [0, 2, 3]], np.uint32)
    away = v + np.float32(1e9)
    scene = I.Scene("quad", away if moving else v, f, np.zeros(2, np.uint32), np.array([[0.5] * 3 + [0.0] * 3], np.float32))
    ctx = gi.Context(width=64, height=64)
    ctx.build_bvh(scene)
    osc = O.OracleScene(scene, use_bvh=False)
    if moving:
        ctx.set_dynamic(v[f].reshape(-1, 9), np.zeros(2, np.uint32))
        osc.set_dynamic(v[f].reshape(-1, 9), np.zeros(2, np.uint32))
    n = len(ALONG)
    o4 = np.zeros((n, 4), np.float32)
    o4[:, axis] = sign * ALONG
    o4[:, b] = np.linspace(-9e6, 9e6, n)
    o4[:, c] = 1e6
    o4[:, 3] = 3.0e38
    d4 = np.zeros((n, 4), np.float32)
    d4[:, c] = -1.0
    d4[:, axis] = 0.0 if sign > 0 else -1e-31      # the reciprocal's sign follows the component's
    tri = torch.zeros(n, dtype=torch.int32, device="cuda")
    t = torch.zeros(n, dtype=torch.float32, device="cuda")
    to, td = torch.from_numpy(o4).cuda(), torch.from_numpy(d4).cuda()
    ctx.trace_rays(to, td, tri, t)
    otri, ot = osc.closest(o4[:, :3].copy(), d4[:, :3].copy())
    assert (otri != 0xFFFFFFFF).all()
    assert np.array_equal(tri.cpu().numpy().view(np.uint32), otri)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), ot.view(np.uint32))
    ctx.trace_rays(to, td, tri, t, any_hit=True)
    assert tri.cpu().numpy().all()
    ctx.close()
