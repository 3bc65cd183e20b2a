"""All iterations in one launch, the frame in its workgroup, against the steps'
launches (eight lanes per pixel): frames of one pixel up to one per thread, and
past what LDS holds; windows of more than one ring; no and wide background
filters; gains and dead pixels.  The two sum a pixel's entries in different
FP32 orders: the bars of the whole-loop tests (1e-3 bins, 2e-5 of intensity)
where the pixel counts agree, and they do but for single pixels."""
import numpy as np
import pytest

from gpu_util import to_dev_hist

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T = 110


@pytest.mark.parametrize("F,rows,cols,kw", [
    (3, 1, 1, {}), (2, 7, 9, {}), (3, 32, 32, {}), (2, 64, 16, {}), (2, 1, 200, {}), (2, 33, 32, {}),
    (2, 24, 20, dict(p_xy=0.8)), (2, 30, 30, dict(p_xy=0.45)), (2, 16, 17, dict(sigma_b=0.0)),
    (2, 20, 20, dict(sigma_b=6.0)), (2, 25, 31, dict(gain=True)), (2, 18, 18, dict(ilp_box=1, n_iter=7)),
])
def test_one_launch_matches_the_steps(F, rows, cols, kw):
    kw = dict(kw)
    with_gain = kw.pop("gain", False)
    rng = np.random.default_rng(rows * 100 + cols)
    i, j = np.meshgrid(np.arange(rows), np.arange(cols), indexing="ij")
    z = rng.poisson(0.01, (F, rows * cols, T))
    for f in range(F):
        for base, share in ((35, 1.0), (70, 0.4)):
            at = (base + 2 * np.sin(0.3 * i + f) + 2 * np.cos(0.25 * j)).reshape(-1)
            for _ in range(8):
                hit = rng.random(rows * cols) < share
                b = np.clip(np.rint(at + rng.normal(0, 1.5, at.shape)), 0, T - 1).astype(int)
                np.add.at(z[f], (np.nonzero(hit)[0], b[hit]), 1)
    hist = to_dev_hist(z.astype(np.uint16).reshape(F, rows, cols, T))
    gain = None
    if with_gain:
        g = rng.uniform(0.5, 2.0, F * rows * cols).astype(np.float32)
        g[::9] = 0.0
        gain = torch.from_numpy(g).cuda()
    res = []
    for fused in (1, 0):
        ctx = rt3d.Context(synth.gaussian_irf(1.5, 9).probs, T, dz=0.1, r_min=0.5, fused_loop=fused, **kw)
        print(f"[gpu-loop-frames] {F} x {rows} x {cols} {kw}, fused_loop {fused}", flush=True)
        o = ctx.reconstruct(hist, gain=gain)
        assert ctx.query().device_error == 0
        res.append((o.pt_off.cpu().numpy().astype(np.int64), o.depth.cpu().numpy(), o.intensity.cpu().numpy(),
                    o.background.cpu().numpy()))
    (pa, da, ra, ba), (pb, db, rb, bb) = res
    same = np.diff(pa) == np.diff(pb)
    assert (~same).sum() <= max(0, same.size // 1000)
    assert np.diff(pa).sum() > 0
    near = same.reshape(F, rows, cols).copy()
    for di in (-1, 0, 1):
        for dj in (-1, 0, 1):
            near &= np.roll(np.roll(same.reshape(F, rows, cols), di, 1), dj, 2)
    for p in np.nonzero(near.reshape(-1) & (np.diff(pa) > 0))[0]:
        n = pa[p + 1] - pa[p]
        assert np.abs(da[pa[p]:pa[p] + n] - db[pb[p]:pb[p] + n]).max() <= 1e-3
        np.testing.assert_allclose(ra[pa[p]:pa[p] + n], rb[pb[p]:pb[p] + n], rtol=2e-5)
    np.testing.assert_allclose(ba, bb, rtol=1e-3, atol=1e-9)
