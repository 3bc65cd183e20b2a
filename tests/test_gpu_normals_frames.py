"""Initial normals of batches of thin and tiny frames, which take a thread per
pixel on the state in memory instead of tiles: the same bits as the same frames
in batches small enough for tiles.  Frames on either side of the lines (4 and
24 pixels a tile), windows of one ring and of four."""
import numpy as np
import pytest

from gpu_util import to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T, IRF = 120, synth.gaussian_irf(1.5, 9)


@pytest.mark.parametrize("p_xy", [1.0, 0.45])
@pytest.mark.parametrize("rows,cols", [(1, 3), (2, 2), (1, 23), (4, 6), (3, 9), (17, 1)])
def test_batches_give_the_same_normals(rows, cols, p_xy):
    F, half = 2600, 1000                     # over 2048 tiles at once, at most 2000 in a part
    rng = np.random.default_rng(rows * 100 + cols)
    i, j = np.mgrid[0:rows, 0:cols]
    d = np.stack([30 + 0.7 * i + 0.4 * j, 70 + 0.5 * j])
    Z = synth.render(rng, IRF, T, np.tile(d.reshape(2, 1, -1), (1, F, 1)), np.full((2, F, rows * cols), 6.0), 0.02)
    off, ent = oracle.compact(Z.reshape(1, F, rows * cols, T))
    ctx = rt3d.Context(IRF.probs, T, dz=0.1, p_xy=p_xy, k_init=3)
    n = rows * cols

    def init(f0, f1):
        o = off[f0 * n:f1 * n + 1].astype(np.int64)
        e = ent[o[0]:o[-1]]
        st = ctx.step(rt3d.STEP_INIT, None, to_dev_u32(o - o[0]), to_dev_u32(np.append(e, 0)), shape=(f1 - f0, rows, cols))
        live = np.arange(4)[:, None] < st.cnt.cpu().numpy()
        return np.where(live, st.n.cpu().numpy(), 0)

    print(f"[gpu-normals-frames] {F} x {rows} x {cols}, p_xy {p_xy}", flush=True)
    whole = init(0, F)
    parts = np.concatenate([init(f, min(f + half, F)) for f in range(0, F, half)], axis=2)
    np.testing.assert_array_equal(whole, parts)
    if min(rows, cols) > 2:                  # (points in one line have no plane: (0, 0, -1))
        assert (np.abs(whole[0]) > 0).mean() > 0.1
