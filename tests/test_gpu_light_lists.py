"""Light lists whose cells keep fewer lights than the list holds (lights out of range or behind the
cell are left out): the cell takes ranks or rounds by the number it keeps, from none to all."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


# 128 and 600 triangles: ranks for cells that keep 12 and 151 of them or more, rounds for the others
@pytest.mark.parametrize("n_lights,k,threshold,shortest,longest", [(64, 256, 0.5, 2, 34), (64, 8, 0.5, 2, 8),
                                                                   (300, 256, 0.15, 104, 215), (300, 256, 1e4, 0, 53)])
def test_lists_shorter_than_their_room(n_lights, k, threshold, shortest, longest):
    pr = _run_stage_parity(I.lights_room_scene(n_lights=n_lights),
                           dict(width=48, height=40, rays_per_probe=8, table_log2=15, light_grid=1, lgrid_k=k,
                                lgrid_dim=5, lgrid_threshold=threshold), [0])
    n = pr.ctx.light_grid()["count"]
    assert n.min() == shortest and n.max() == longest
