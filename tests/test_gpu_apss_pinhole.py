"""The pinhole camera's APSS step against the oracle where its tiles, windows
and point lists change form: frames of one pixel up to several tiles with
remainders, window radii 1 to 5, fields of view up to 150 degrees (windows cut
to narrow slanted ellipses), surfaces from the camera's own place (window
never cut) to far ones (the pixel alone), up to four points per pixel, isolated
points, a pixel without any.  The bar is the one of the step's other tests
(1e-3 bins and normal components)."""
import numpy as np
import pytest

from gpu_util import device_to_oracle, oracle_to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

T, DZ = 1200, 0.1


def state(rng, F, rows, cols, persp, depths):
    """Smooth surfaces at the given depths (bins), each over most of the
    pixels, and isolated points between them."""
    s = oracle.State(F, rows, cols, 4)
    i, j = np.meshgrid(np.arange(rows), np.arange(cols), indexing="ij")
    for f in range(F):
        for q in range(rows * cols):
            t = [d + 2.0 * np.sin(0.21 * i.flat[q] + k) + 1.5 * np.cos(0.17 * j.flat[q] - f) + rng.normal(0, 0.3)
                 for k, d in enumerate(depths) if rng.random() < 0.8]
            if rng.random() < 0.05 and len(t) < 4:
                t.append(rng.uniform(900, 1100))
            t = np.sort(np.clip(t, 0.0, T - 1.0))
            p = f * rows * cols + q
            s.cnt[p] = len(t)
            s.t[p, :len(t)] = t
            s.r[p, :len(t)] = 1.0
            v = np.array([persp * (j.flat[q] - 0.5 * (cols - 1)), persp * (i.flat[q] - 0.5 * (rows - 1)), 1.0])
            n = -v[None, :] / np.linalg.norm(v) + rng.normal(0, 0.2, (len(t), 3))
            s.n[p, :len(t)] = n / np.linalg.norm(n, axis=1, keepdims=True)
    return s


@pytest.mark.parametrize("F,rows,cols,persp,p_xy,depths", [
    (1, 1, 1, 0.05, 0.41, (300.0,)),
    (2, 16, 16, 0.02, 0.41, (200.0, 500.0)),
    (1, 17, 33, 0.02, 0.5, (200.0, 300.0, 760.0)),
    (2, 5, 47, 0.15, 0.41, (120.0, 400.0)),
    (1, 61, 3, 0.12, 0.41, (60.0, 100.0, 150.0, 300.0)),
    (1, 33, 31, 0.02, 2.0, (100.0, 160.0)),
    (1, 20, 20, 0.002, 0.41, (4.0, 60.0, 700.0)),
    (1, 18, 18, 0.03, 1.0, (900.0, 1000.0)),
])
def test_pinhole_apss_matches_oracle(F, rows, cols, persp, p_xy, depths):
    rng = np.random.default_rng(rows * 100 + cols)
    irf = synth.gaussian_irf(1.5, 9).probs
    p = dict(dz=DZ, p_xy=p_xy, persp=persp)
    s0 = state(rng, F, rows, cols, persp, depths)
    print(f"[gpu-apss-pinhole] {F}x{rows}x{cols} persp {persp} p_xy {p_xy}: {int(s0.cnt.sum())} points", flush=True)
    so = oracle.Oracle(oracle.Model(irf, T), oracle.Params(**p)).apss(s0.copy())
    sg = device_to_oracle(rt3d.Context(irf, T, **p).step(rt3d.STEP_APSS, oracle_to_device(s0)), 4)
    np.testing.assert_array_equal(sg.cnt, so.cnt)
    live = np.arange(4)[None, :] < s0.cnt[:, None]
    assert np.abs(sg.t - so.t)[live].max(initial=0.0) <= 1e-3
    assert np.abs(sg.n - so.n)[live].max(initial=0.0) <= 1e-3
