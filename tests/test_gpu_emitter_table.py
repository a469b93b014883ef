"""Emitter tables below and above 64 KB, uploaded with the moving lights at every frame: rays, light
samples and cell sums against the oracle while the lights move, appear and go."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2310_19855_amd import inputs as I  # noqa: E402
from test_gpu_parity import _run_stage_parity  # noqa: E402


def _scene(n):
    """the room with n small emissive triangles in the air; 0, 2 and 64 moving ones, by frame"""
    room = I.room_scene()
    rng = np.random.default_rng(n)
    v = (rng.uniform(1.0, 2.5, (n, 1, 3)) + rng.uniform(-0.02, 0.02, (n, 3, 3))).astype(np.float32).reshape(-1, 3)
    f = len(room.verts) + np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)
    glow = np.uint32(np.argmax(room.materials[:, 3]))

    def lights(frame):
        k = (2, 64, 0, 1)[frame % 4]
        r = np.random.default_rng(frame)
        tv = r.uniform(2.6, 2.9, (k, 9)).astype(np.float32)
        return tv, np.full(k, glow, np.uint32)
    return I.Scene("room", np.concatenate([room.verts, v]), np.concatenate([room.idx, f]),
                   np.concatenate([room.tri_mat, np.full(n, glow, np.uint32)]), room.materials, dynamic=lights)


# 56 bytes an entry: 1,100 pass 64 KB with the 64 moving lights alone; 6,000 are 336 KB
@pytest.mark.parametrize("n", [1, 1100, 6000])
def test_tables_of_every_size(n):
    _run_stage_parity(_scene(n), dict(width=64, height=48, rays_per_probe=16, table_log2=16), [0, 1, 2, 3])
