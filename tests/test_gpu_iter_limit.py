"""Around the lines up to which an iteration takes three launches on tiles: the
batches on either side, full tiles and thin ones, give the same bits as a context
whose background filter is timed, which runs the steps one by one."""
import numpy as np
import pytest

from gpu_util import to_dev_hist

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1905_06700_amd import rt3d, synth  # noqa: E402
from test_gpu_iter_tiles import T, photons  # noqa: E402


# frames, rows, cols: 2560, 2720, 2752 full tiles; columns of 2048 and 2049 tiles;
# a row of 2125; one-pixel frames, 2720 and 2721 tiles
@pytest.mark.parametrize("F,rows,cols", [(80, 32, 32), (85, 32, 32), (86, 32, 32), (1, 8192, 1), (1, 8193, 1),
                                         (1, 1, 17000), (2720, 1, 1), (2721, 1, 1)])
def test_both_sides_equal_the_steps(F, rows, cols):
    rng = np.random.default_rng(F + rows)
    z = photons(rng, [(F * rows, cols)])
    hist = to_dev_hist(z)
    res = []
    for timed in (None, "bfilter"):
        ctx = rt3d.Context(synth.gaussian_irf(1.5, 9).probs, T, dz=0.1, r_min=0.05, r_init=0, fused_loop=0, n_iter=2)
        ctx.profile(timed)
        ctx.workspace(F, rows, cols, int(z.sum()) + 1)
        out = ctx.make_output(z.shape[0])
        print(f"[gpu-iter-limit] {F} x {rows} x {cols} {'steps' if timed else 'as ruled'}", flush=True)
        ctx.reconstruct_into(out, F, rows, cols, hist=hist)
        assert ctx.query().device_error == 0
        n = int(out.pt_off[-1].item())
        assert n > z.shape[0] // 2
        res.append([x.cpu().numpy() for x in (out.pt_off, out.background, out.depth[:n], out.intensity[:n], out.normal[:n])])
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)
