"""The reservoir table and the light lists where their kernels take another path: cells that lose
their bidding place to another cell (a small table holding many cells), one ray and one cell, lists
made by ranks and by rounds, lists longer than the lights there are."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


@pytest.mark.parametrize("W,H,rays,cell_scale,log2", [(96, 64, 33, 1.2, 9), (8, 8, 1, 10.0, 12), (100, 76, 64, 10.0, 17)])
def test_reservoirs_of_crowded_and_empty_tables(W, H, rays, cell_scale, log2):
    _run_stage_parity(I.lights_room_scene(n_lights=16), dict(width=W, height=H, rays_per_probe=rays, table_log2=17,
                                                             cell_scale=cell_scale, light_grid=1, lgrid_k=32, restir=1,
                                                             restir_log2=log2), [0, 1, 2])


@pytest.mark.parametrize("n_lights,k", [(1, 1), (16, 256), (64, 1), (64, 100), (300, 4), (300, 256)])
def test_light_lists_by_ranks_and_rounds(n_lights, k):
    """2 to 600 emitter triangles; ranks are taken where 3 n (n/64 + 1) is below K (3 (n/64 + 1) + 90)"""
    _run_stage_parity(I.lights_room_scene(n_lights=n_lights), dict(width=48, height=40, rays_per_probe=8, table_log2=15,
                                                                   light_grid=1, lgrid_k=k, lgrid_dim=5), [0])
