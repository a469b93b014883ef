"""The gradient pairs of a training step are sorted either by their full key or level by level
(where that saves a pass and a level's pairs fill whole sort tiles): both sides of that rule
against the float64 oracle, level by level."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from oracle import learned as OL  # noqa: E402
from test_gpu_learned import SEED, _cos, _ctx, _samples, _unpack  # noqa: E402


def _bf16(x):
    return torch.from_numpy(np.asarray(x, np.float32)).bfloat16().float().numpy().astype(np.float64)


def _grid_gradient(spec, p, x32, nrm, tgt, S=128.0):
    """the oracle's grid gradient with every matrix operand rounded to BF16 (a unit that BF16 puts
    on the other side of zero turns one level's small gradient by up to 4 degrees)"""
    _, c = OL.forward(spec, p, x32, nrm)
    W1, W2, W3 = _bf16(p["W1"]), _bf16(p["W2"]), _bf16(p["W3"])
    z1 = _bf16(c["X"]) @ W1.T
    z2 = _bf16(np.maximum(z1, 0)) @ W2.T
    y = (_bf16(np.maximum(z2, 0)) @ W3.T)[:, :3]
    dy = np.zeros((len(y), 16))
    dy[:, :3] = _bf16(2 * (y - tgt) / (y * y + 0.01) / (3 * len(y)) * S) / S
    dX = _bf16((_bf16((dy @ W3) * (z2 > 0)) @ W2) * (z1 > 0)) @ W1
    g = np.zeros_like(p["grid"])
    for l, (idx, w) in enumerate(c["corners"]):
        for f in range(2):
            np.add.at(g[l][:, f], idx.ravel(), (w * dX[:, 2 * l + f][:, None]).ravel())
    return g


# by level: one tile per level and one digit (11 x 2^8); two digits of which the second is short
# (2 x 2^16 has 16 bits against 17; 16 x 2^13); levels that are no multiple of 8 (5 x 2^7).
# Full key: half a tile per level (16 x 2^13 at 2^7 samples); no pass saved (16 x 2^10).
@pytest.mark.parametrize("levels,tlog2,blog2", [(11, 8, 8), (2, 16, 8), (16, 13, 10), (5, 7, 9), (16, 13, 7),
                                                (16, 10, 8)])
def test_every_level_gets_its_own_gradient(levels, tlog2, blog2):
    """Pairs that went to another level or entry, or were lost at a tile's edge, would turn that
    level's gradient (the bounds are the ones the whole gradient is held to)."""
    spec = OL.Spec(levels=levels, table_log2=tlog2)
    ctx, sc, lo, hi = _ctx(mlp_levels=levels, mlp_table_log2=tlog2, mlp_batch_log2=blog2)
    pos, nrm, tgt = _samples(1 << blog2, lo, hi, seed=blog2)
    tp, tn, tt = (torch.from_numpy(a).cuda() for a in (pos, nrm, tgt))
    ctx.learned_step(tp, tn, tt, apply=False)
    torch.cuda.synchronize()
    got = _unpack(ctx, spec)["grid_g"].reshape(levels, spec.T, 2) / 128.0
    x32 = OL.normalize_pos(pos[:, :3], lo, hi)
    g = _grid_gradient(spec, OL.init_params(spec, SEED), x32, nrm[:, :3], tgt[:, :3])
    for l in range(levels):
        ref = g[l]
        assert _cos(got[l], ref) > 0.999, l
        assert abs(np.linalg.norm(got[l]) / np.linalg.norm(ref) - 1) < 0.01, l
        assert not got[l][(ref == 0).all(1)].any(), l
    ctx.close()


@pytest.mark.parametrize("counts", [(1024,), (700, 90, 33, 201), (63, 64, 65, 128, 192, 255, 257), (1, 1023)])
def test_long_runs_of_one_entry_sum_over_tiles(counts):
    """Samples in a few points: an entry's pairs run over parts of one 256-pair tile, all of it,
    and several, so that a tile's last entry begins in each of its four runs of 64 or before it."""
    levels, tlog2, blog2 = 4, 12, 10
    assert sum(counts) <= 1 << blog2
    spec = OL.Spec(levels=levels, table_log2=tlog2)
    ctx, sc, lo, hi = _ctx(mlp_levels=levels, mlp_table_log2=tlog2, mlp_batch_log2=blog2)
    pos, nrm, tgt = _samples(1 << blog2, lo, hi, seed=len(counts))
    at = 0
    for c in counts:
        pos[at:at + c] = pos[at]
        at += c
    tp, tn, tt = (torch.from_numpy(a).cuda() for a in (pos, nrm, tgt))
    ctx.learned_step(tp, tn, tt, apply=False)
    torch.cuda.synchronize()
    got = _unpack(ctx, spec)["grid_g"].reshape(levels, spec.T, 2) / 128.0
    x32 = OL.normalize_pos(pos[:, :3], lo, hi)
    g = _grid_gradient(spec, OL.init_params(spec, SEED), x32, nrm[:, :3], tgt[:, :3])
    for l in range(levels):
        assert _cos(got[l], g[l]) > 0.999, l
        assert abs(np.linalg.norm(got[l]) / np.linalg.norm(g[l]) - 1) < 0.01, l
    ctx.close()
