"""The denoiser's two passes where they can go wrong: squares cut by the image edge, windows wider
than the image, every pixel in the wide or the narrow class, the image filtered in place, and a
captured call that must go on from the history the replay before it left."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from gpu_common import assert_close  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402


def _irradiance(H, W, prim, frame):
    """seeded irradiance with flags: 2 (no probe) here and there, 3 on sky"""
    rng = np.random.default_rng(100 + frame)
    e = rng.uniform(0.0, 3.0, (H, W, 4)).astype(np.float32)
    e[..., 3] = np.where(rng.random((H, W)) < 0.1, 2.0, 0.0)
    sky = prim == 0xFFFFFFFF
    e[sky] = (0.0, 0.0, 0.0, 3.0)
    return e


@pytest.mark.parametrize("W,H,radius,scene", [(8, 8, 16, "room"), (17, 33, 4, "room"), (50, 16, 1, "field"),
                                              (33, 47, 16, "field")])
def test_denoiser_edges_and_radii(W, H, radius, scene):
    sc = I.room_scene() if scene == "room" else I.field_scene(n_boxes=300, n_spheres=2)
    cfg = dict(O.default_config(), width=W, height=H, denoise=1, dn_hist_max=4, dn_radius=radius)
    osc = O.OracleScene(sc)
    ost = O.OracleFrameState(osc, cfg)
    dn = gi.Denoiser(W, H, hist_max=4, radius_max=radius)
    for f in range(5):
        fr = I.room_camera(0) if scene == "room" else I.orbit_camera(3 * f)
        fr.index = f
        pos, nrm, _, prim = osc.gbuffer(fr, W, H)
        prim = prim.reshape(H, W)
        e = _irradiance(H, W, prim, f)
        dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pos.reshape(H, W, 4), nrm.reshape(H, W, 4),
                                                                         prim.view(np.int32), e)]
        dn(fr, dev[0], dev[1], dev[2], dev[3], dev[3])            # in place
        ref = ost.denoise(fr, pos, nrm, prim, e)
        gh, grad = dn.state()
        oh, orad = ost.denoise_state()
        assert np.array_equal(gh[..., 3], oh[..., 3]) and np.array_equal(grad, orad)
        assert_close(gh[..., :3], oh[..., :3], what="history")
        got = dev[3].cpu().numpy()
        assert np.array_equal(got[..., 3], ref[..., 3])
        assert_close(got[..., :3], ref[..., :3], what="denoised irradiance")
    dn.close()


def test_replayed_denoiser_goes_on_from_its_history():
    W, H, n = 40, 24, 6
    osc = O.OracleScene(I.room_scene())
    fr = I.room_camera(0)
    pos, nrm, _, prim = osc.gbuffer(fr, W, H)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (pos.reshape(H, W, 4), nrm.reshape(H, W, 4),
                                                                     prim.reshape(H, W).view(np.int32))]
    e = [torch.from_numpy(_irradiance(H, W, prim.reshape(H, W), f)).cuda() for f in range(n)]
    eager, replayed = gi.Denoiser(W, H), gi.Denoiser(W, H)
    want, got, irr = torch.zeros_like(e[0]), torch.zeros_like(e[0]), e[0].clone()
    eager(fr, *dev, e[0], want)
    replayed(fr, *dev, irr, got)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        replayed(fr, *dev, irr, got)
    for f in range(1, n):
        eager(fr, *dev, e[f], want)
        irr.copy_(e[f])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(want, got), f"replay {f}"
        (wh, wr), (gh, gr) = eager.state(), replayed.state()
        assert np.array_equal(wh, gh) and np.array_equal(wr, gr), f"state after replay {f}"
    eager.close()
    replayed.close()
