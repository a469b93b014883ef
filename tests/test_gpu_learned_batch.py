"""Training batches of more than 32 sort tiles (65,536 rows), whose grouping takes scanned tile
counts, against a stable host sort by the rows' Morton codes; 32 tiles, where it adds them up itself,
beside them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import learned as OL  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402

SMALL = dict(cache_mode=gi.CACHE_MLP_BF16, mlp_levels=2, mlp_table_log2=8)


def _assert_grouped(b, sc):
    order = OL.group_order(OL.normalize_pos(b["raw"][:, 0, :3], sc.verts.min(0), sc.verts.max(0)))
    assert np.array_equal(b["grouped"].view(np.uint32), b["raw"][order].view(np.uint32))


# 40 tiles, 33 whole ones, 32 and one of 128 rows, 64 tiles in one step; 32
@pytest.mark.parametrize("blog2,steps", [(14, 5), (11, 33), (7, 513), (17, 1), (14, 4)])
def test_frame_batches(blog2, steps):
    sc = I.room_scene()
    ctx = gi.Context(width=256, height=256, rays_per_probe=32, table_log2=16, mlp_batch_log2=blog2, mlp_steps=steps,
                     **SMALL)
    ctx.build_bvh(sc)
    gb = gi.GBuffer(256, 256)
    fr = I.room_camera(0)
    ctx.render_gbuffer(fr, gb.pos, gb.nrm, gb.alb, gb.prim)
    ctx.spawn_probes(fr, gb.pos, gb.nrm, gb.prim)
    ctx.trace_probes(fr)
    ctx.learned_train(fr)
    b = ctx.learned_batch()
    assert len(b["raw"]) == steps << blog2
    # the picks: rays of the training list at the frame's stratified places, in ray order
    ray = np.unique(b["gid"])
    assert 1 < len(ray) <= b["n_train"] <= 32 * 32 * 32 and (np.diff(b["gid"].astype(np.int64)) >= 0).all()
    rec = ctx.rays()
    assert np.array_equal(b["raw"][:, 0, 3].view(np.uint32), rec["t"][b["gid"]].view(np.uint32))
    _assert_grouped(b, sc)
    ctx.close()


@pytest.mark.parametrize("blog2", [16, 17])
def test_caller_batches(blog2):
    sc = I.room_scene()
    ctx = gi.Context(width=64, height=64, mlp_batch_log2=blog2, mlp_steps=1, **SMALL)
    ctx.build_bvh(sc)
    rng = np.random.default_rng(blog2)
    n = 1 << blog2
    rows = rng.normal(size=(n, 3, 4)).astype(np.float32)
    rows[:, 0, :3] = rng.uniform(sc.verts.min(0), sc.verts.max(0), (n, 3))
    rows[:, 2] = np.abs(rows[:, 2])
    ctx.learned_step(*(torch.from_numpy(np.ascontiguousarray(rows[:, k])).cuda() for k in range(3)), apply=False)
    b = ctx.learned_batch()
    assert np.array_equal(b["raw"].view(np.uint32), rows.view(np.uint32))
    _assert_grouped(b, sc)
    ctx.close()
