"""Two cells of one bucket and one fingerprint share a reservoir slot: it holds the reservoir (and
the cell) of the lowest ray id that offers to it, whichever of the two cells that ray hit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle as O  # noqa: E402
from gpu_common import Pair, bits  # noqa: E402
from paper_2310_19855_amd import gi  # noqa: E402
from paper_2310_19855_amd import inputs as I  # noqa: E402

CELLS = ((16, 52, 109), (17, 4, 110))     # same fingerprint, and same bucket of up to 128
SIDE, W, H, RAYS = 0.1, 16, 8, 16


def _hashes(cell):
    lo, hi = (cell[0] | cell[1] << 18) & 0xFFFFFFFF, cell[1] >> 14 | cell[2] << 4
    return O.pcg((lo + O.pcg(hi)) & 0xFFFFFFFF), O.xxh32((lo + O.xxh32(hi)) & 0xFFFFFFFF)


def _scene():
    """a patch inside each of the two cells, facing up, under one light that faces down"""
    v, f, m = [], [], []
    for k, cell in enumerate(CELLS + (None,)):
        x, y, z = (1.7, 8.0, 11.0) if cell is None else (np.array(cell) + 0.5) * SIDE
        h = 1.0 if cell is None else 0.04
        q = [(x - h, y, z - h), (x - h, y, z + h), (x + h, y, z + h), (x + h, y, z - h)]
        v += q if cell is not None else q[::-1]
        f += [(4 * k, 4 * k + 1, 4 * k + 2), (4 * k, 4 * k + 2, 4 * k + 3)]
        m += [int(cell is None)] * 2
    return I.Scene("patches", np.array(v, np.float32), np.array(f, np.uint32), np.array(m, np.uint32),
                   np.array([[0.5, 0.5, 0.5, 0, 0, 0], [0, 0, 0, 9.0, 5.0, 2.0]], np.float32))


@pytest.mark.parametrize("order", [(0, 1), (1, 0)])
@pytest.mark.parametrize("log2", [6, 12])
def test_cells_of_one_slot_keep_the_lowest_ray(order, log2):
    (b0, f0), (b1, f1) = (_hashes(c) for c in CELLS)
    assert f0 == f1 and b0 % 128 == b1 % 128
    pr = Pair(_scene(), dict(width=W, height=H, rays_per_probe=RAYS, table_log2=10, cell_scale=1.0 / SIDE,
                             light_grid=1, restir=1, restir_log2=log2))
    # one probe 5 mm above each patch, looking down on it
    pos = np.zeros((H, W, 4), np.float32)
    nrm = np.zeros((H, W, 4), np.float32)
    nrm[..., 1] = -1.0
    for tile, k in enumerate(order):
        pos[:, 8 * tile:8 * tile + 8, :3] = (np.array(CELLS[k]) + 0.5) * SIDE + (0.0, 0.005, 0.0)
    prim = np.zeros((H, W), np.uint32)
    dp, dn, dprim = (torch.from_numpy(a).cuda() for a in (pos, nrm, prim.view(np.int32)))
    for frame in range(3):
        fr = I.room_camera(0)
        fr.index = frame
        pr.ctx.spawn_probes(fr, dp, dn, dprim)
        pr.ost.spawn(fr, pos, nrm, prim)
        pr.ctx.trace_probes(fr)
        pr.ost.trace(fr)
        rays, gr = pr.ost.rays(), pr.ctx.rays()
        assert np.array_equal(gr["tri"], rays["tri"])
        hit = (rays["cell"] & gi.RAY_HIT) != 0
        for tile, k in enumerate(order):          # both cells are offered to
            assert np.isin(rays["tri"][hit & (np.arange(2 * RAYS) // RAYS == tile)], (2 * k, 2 * k + 1)).any()
        got, ref = pr.ctx.reservoirs(), pr.ost.reservoirs()
        c = CELLS[order[0]]
        assert c[0] | c[1] << 18 | c[2] << 36 in ref["key"].tolist()
        for k in ("id", "key", "k", "M"):
            assert np.array_equal(got[k], ref[k]), (frame, k)
        for k in ("y", "W", "n"):
            assert np.array_equal(bits(got[k]), bits(ref[k].astype(np.float32))), (frame, k)
        pr.ctx.cache_update(fr)
        pr.ost.update(fr)
