"""The dense search's weights at their widest: 13 and 14 bits of rest in two
digits (sbr_guess raises the weights), and past them (the search from the
lists).  Counts and depths equal to the oracle's, the rest to the rounding of
the stored values."""
import numpy as np
import pytest

from gpu_util import device_to_oracle, to_dev_u32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402
from paper_1905_06700_amd import rt3d, synth  # noqa: E402

IRF, T, ROWS, COLS = synth.gaussian_irf(1.5, 9), 4613, 8, 9


@pytest.mark.parametrize("sbr_guess", [1.0, 1500.0, 1e5, 1e9, 1e11, 1e13])
def test_weights_of_any_size(sbr_guess):
    rng = np.random.default_rng(5)
    i, j = np.mgrid[0:ROWS, 0:COLS].astype(np.float64)
    d = 0.1 * T + 0.8 * T * (j + 0.3 * i) / (COLS + 0.3 * ROWS)
    Z = synth.render(rng, IRF, T, d[None], rng.uniform(5.0, 11.0, (1, ROWS, COLS)), 30.0 / T)
    p = dict(dz=0.1, p_xy=1.0, r_min=1.0, r_init=1, k_init=3, sbr_guess=sbr_guess)
    off, ent = oracle.compact(Z[None])
    so = oracle.Oracle(oracle.Model(IRF.probs, T), oracle.Params(**p)).init(off, ent, oracle.State(1, ROWS, COLS, 4))
    print(f"[gpu-init-digits] sbr_guess {sbr_guess}", flush=True)
    ctx = rt3d.Context(IRF.probs, T, **p)
    sg = device_to_oracle(ctx.step(rt3d.STEP_INIT, None, to_dev_u32(off), to_dev_u32(np.append(ent, 0)), shape=(1, ROWS, COLS)), 4)
    assert so.cnt.sum() > 0
    np.testing.assert_array_equal(sg.cnt, so.cnt)
    np.testing.assert_array_equal(sg.t, so.t)
    np.testing.assert_allclose(sg.r, so.r, rtol=1e-6, atol=1e-6)
    np.testing.assert_allclose(sg.b, so.b, rtol=1e-6, atol=1e-12)
