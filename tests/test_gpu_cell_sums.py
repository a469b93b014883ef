"""Fixed-point cell sums that pass 2^32: two words share one 64-bit addition, whose carries must
not be seen.  A light so bright that lit samples are clamped, the largest fixed-point scale, and
cells large enough to collect hundreds of samples: sums, wrap count and everything after them
against the oracle."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


@pytest.mark.parametrize("light,cell_scale,tiles", [(1e6, 0.5, 0), (1e6, 4.0, 0), (2e3, 0.5, 0), (1e6, 4.0, 1)])
def test_sums_that_wrap_equal_the_oracle(light, cell_scale, tiles):
    pr = _run_stage_parity(I.room_scene(light_le=light), dict(width=128, height=96, rays_per_probe=64, table_log2=14,
                                                              cell_scale=cell_scale, frac_bits=16, r_max=1000.0,
                                                              cache_tiles=tiles), [0, 1])
    if light > 1e5 and cell_scale < 1.0:   # clamped samples in 2 m cells; the other inputs stay below 2^32
        assert pr.ctx.stats()["wraps"] > 0
