"""State that frames hand on, at the sizes and histories where its kernels change path: the list of
override tiles over more than one round and with a part of a group at the end; two-level cache
tiles that rest, are only looked up, age out and come back."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


@pytest.mark.parametrize("width,height", [(40, 24), (1000, 76), (2104, 1000)])
def test_override_list_lengths(width, height):
    """15, 1,250 and 32,875 tiles (one list round holds 32,768)"""
    _run_stage_parity(I.room_scene(), dict(width=width, height=height, rays_per_probe=1, table_log2=16, temporal=1,
                                           upscale=2), [0, 1, 2])


@pytest.mark.parametrize("bounces,max_life", [(1, 3), (2, 2)])
def test_tiles_rest_age_out_and_return(bounces, max_life):
    """two cameras in turn: the tiles one sees rest while the other looks elsewhere"""
    _run_stage_parity(I.room_scene(), dict(width=96, height=64, rays_per_probe=16, table_log2=10, cache_tiles=1,
                                           bounces=bounces, max_life=max_life), [0, 1, 2, 3, 4, 5],
                      camera=lambda f: I.room_camera(0, seed=2 + (f // 2) % 2))
